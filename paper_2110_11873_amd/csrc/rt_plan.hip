// rt_plan.hip -- launch plans of the sweep (host code): the rays of a slab, their
// chunks and wave-batches, the tile-ordered coefficients' layout, and the block
// lists of the sweeps.
#include <algorithm>
#include <cmath>
#include <string>
#include <utility>
#include <vector>

#include "rt_internal.h"

namespace rt {

namespace {

std::string slab_name(long long i) { return "ns[" + std::to_string(i) + "]"; }

int chunks_for(int ns, int L) {
    const int x = ns - 1;
    int C = kMinChunks;
    while (C < kWave && C * L < x) C <<= 1;
    return C;
}

// The tile geometry of one slab for a plan of longest chunk L: chunks per
// ray, chunk length, long chunks, rays per wave-batch, wave-batches per
// direction and tile entries per wave-batch.
struct SlabTiles {
    int C, Leff, nlong, G, nwb, bstride;
};
SlabTiles slab_tiles(int ns, int L, int n_nu) {
    SlabTiles t;
    t.C = chunks_for(ns, L);
    t.Leff = chunk_len(ns, t.C, L);
    // chunk lengths Leff and Leff - 1 tile the ns - 1 intervals exactly
    // when Leff is ceil((ns - 1) / C); otherwise (lengths rounded up to
    // a compiled one) all chunks are long and the last ones end past the
    // slab's bottom in identity steps
    t.nlong = t.C;
    if (chunk_len_step(L) == 1) {
        const int r = (ns - 1) - t.C * (t.Leff - 1);
        if (r >= 1 && r <= t.C) t.nlong = r;
    }
    t.G = kWave / t.C;
    t.nwb = (n_nu + t.G - 1) / t.G;
    t.bstride = (t.Leff - 1) * kWave + (t.G * t.nlong + 15) / 16 * 16;
    return t;
}

// Frequencies of a slab whose opacity ratios agree to kSameOpac share a formal
// solution: under complete redistribution the source does not depend on
// frequency and a ray sees it only through kappa = r_p / |mu|, so their
// weights w_p phi_p add.  The group's opacity is the weighted mean, which
// cancels the first-order difference; the second is below 1e-24.  A line
// profile that is even about its centre halves the rays this way (the two
// halves of a computed grid differ by up to 1.5e-14); without equal opacities
// every group is one frequency.  512 slabs of 101 frequencies: the FP64
// operator takes 250 us with a ray per frequency, 140 us with one per opacity.
// Every slab gets the same number of rays (the largest count), the rest with
// weight zero: one uneven profile has the whole batch swept ray by ray.
// Strongest opacity first.  The order sets that of the additions and nothing
// else; this one was kept because GMRES restarted every 2 steps on an
// ill-conditioned slab, whose step count moves between 157 and 312 when tau is
// perturbed by 1e-16, came nearer the oracle's own count with it (203 against
// 159 with the weakest first, the oracle's 248).
constexpr double kSameOpac = 1e-12;
bool same_opacity(double first, double x) { return x - first <= kSameOpac * first; }

int merge_frequencies(const rt_problem *p, std::vector<double> &opac, std::vector<double> &wphi) {
    const int n = p->n_nu;
    std::vector<std::pair<double, double>> f(n);  // (opacity, weight)
    std::vector<double> kap((size_t)p->n_atm * n), w((size_t)p->n_atm * n);
    std::vector<int> count(p->n_atm, 0);
    int most = 0;
    for (int a = 0; a < p->n_atm; ++a) {
        const double *op = p->opac + (long long)a * n, *ph = p->phi + (long long)a * n;
        for (int q = 0; q < n; ++q) f[q] = {op[q], p->w_nu[q] * ph[q]};
        std::sort(f.begin(), f.end());
        int g = 0;
        for (int i = 0; i < n; ++g) {
            const double first = f[i].first;
            double sw = 0.0, excess = 0.0;  // of the opacity over the first's
            for (; i < n && same_opacity(first, f[i].first); ++i) {
                sw += f[i].second;
                excess += f[i].second * (f[i].first - first);
            }
            kap[(size_t)a * n + g] = sw > 0.0 ? first + excess / sw : first;
            w[(size_t)a * n + g] = sw;
        }
        count[a] = g;
        most = std::max(most, g);
    }
    opac.resize((size_t)p->n_atm * most);
    wphi.resize((size_t)p->n_atm * most);
    for (int a = 0; a < p->n_atm; ++a)
        for (int g = 0; g < most; ++g) {
            const bool on = g < count[a];
            const size_t e = (size_t)a * n + (on ? count[a] - 1 - g : 0);
            opac[(size_t)a * most + g] = kap[e];
            wphi[(size_t)a * most + g] = on ? w[e] : 0.0;
        }
    return most;
}

// Longest blocks first (work ~ wave-batches x chunk length, the same lane count
// per batch); ties keep slab order.
void order_blocks(std::vector<BlockDesc> &list, const std::vector<AtmDesc> &atm) {
    std::stable_sort(list.begin(), list.end(), [&](const BlockDesc &x, const BlockDesc &y) {
        return (long long)x.wb_count * atm[x.atm].Leff > (long long)y.wb_count * atm[y.atm].Leff;
    });
    // XCD-aware order: workgroups are handed to the 8 XCDs in turn by
    // index, and the blocks of one slab stage the same sources, so each
    // slab's run of blocks goes to one XCD (indices 8 apart, one L2) and
    // consecutive runs to consecutive XCDs -- the longest-first order
    // kept per group of 8 runs.  Applied when the runs fill the XCDs
    // evenly (equal-size runs, a multiple of 8 of them).
    constexpr int kXcd = 8;
    std::vector<std::vector<BlockDesc>> q(kXcd);
    size_t i = 0;
    int run = 0;
    while (i < list.size()) {
        size_t j = i;
        while (j < list.size() && list[j].atm == list[i].atm) ++j;
        for (size_t k = i; k < j; ++k) q[run % kXcd].push_back(list[k]);
        ++run;
        i = j;
    }
    bool even = true;
    for (int x = 1; x < kXcd; ++x) even = even && q[x].size() == q[0].size();
    if (even && !q[0].empty()) {
        std::vector<BlockDesc> out;
        out.reserve(list.size());
        for (size_t k = 0; k < q[0].size(); ++k)
            for (int x = 0; x < kXcd; ++x) out.push_back(q[x][k]);
        list.swap(out);
    }
}

// The block list over the slabs `atm` (geometry set) of M directions, for blocks
// of W waves, wpd per direction, each with nb[a] wave-batches of slab a.
SweepPlan make_plan(const std::vector<AtmDesc> &atm, int M, int W, int wpd,
                    const std::vector<int> &nb) {
    SweepPlan pl;
    pl.wpd = wpd;
    pl.atm = atm;
    const int dpb = W / wpd;  // directions per block
    const int dgroups = (M + dpb - 1) / dpb;
    for (size_t a = 0; a < atm.size(); ++a) {
        AtmDesc &d = pl.atm[a];
        const int wb_per_block = wpd * nb[a];
        const int blk_per_dir = (d.nwb + wb_per_block - 1) / wb_per_block;
        d.nblk = dgroups * blk_per_dir;
        d.blk_first = pl.n_blocks;
        d.part_off = pl.n_partial;
        for (int mg = 0; mg < dgroups; ++mg)
            for (int bb = 0; bb < blk_per_dir; ++bb) {
                BlockDesc bd{};
                bd.atm = (int)a;
                bd.m = mg * dpb;
                bd.wb_first = bb * wb_per_block;
                bd.wb_count = std::min(wb_per_block, d.nwb - bd.wb_first);
                bd.slot = mg * blk_per_dir + bb;
                bd.wpd = wpd;
                pl.blk.push_back(bd);
            }
        pl.n_blocks += d.nblk;
        pl.nblk_max = std::max(pl.nblk_max, d.nblk);
        pl.n_partial += (long long)d.nblk * 2 * d.ns;
    }
    order_blocks(pl.blk, pl.atm);
    return pl;
}

}  // namespace

int distinct_opacities(const rt_problem *p) {
    if (!p->opac || p->n_nu < 1) return 0;
    int most = 0;
    std::vector<double> f(p->n_nu);
    for (int a = 0; a < p->n_atm; ++a) {
        std::copy_n(p->opac + (long long)a * p->n_nu, p->n_nu, f.begin());
        for (double x : f)
            if (!std::isfinite(x) || !(x > 0.0)) return 0;
        std::sort(f.begin(), f.end());
        int g = 0;
        for (size_t i = 0; i < f.size(); ++g) {
            const double first = f[i];
            while (i < f.size() && same_opacity(first, f[i])) ++i;
        }
        most = std::max(most, g);
    }
    return most;
}

// Chunk length: the largest L whose lane count fills the chip (about two
// waves per SIMD) -- longer chunks mean fewer scan steps and partial sums --
// else the shortest, for the most parallelism on small problems.
int auto_chunk(const std::vector<int> &ns, int rays) {
    const long long target = 256LL * 4 * kWave * 2;
    int best = 4;
    for (int L : {4, 8}) {
        bool fits = true;
        long long lanes = 0;
        for (int n : ns) {
            const int C = chunks_for(n, L);
            if ((long long)C * L < n - 1) fits = false;
            lanes += (long long)rays * C;
        }
        if (fits && lanes >= target) best = L;
    }
    // a slab deeper than 64 * best intervals needs longer chunks
    for (int n : ns)
        while (best < 32 && (long long)kWave * best < n - 1) best *= 2;
    return best;
}

// The sweep addresses the tiles of one (slab, direction) through 32-bit
// buffer offsets, in entries of up to 16 bytes (FP64 pairs): reject plans
// whose tiles of one direction exceed 2^31 - 1 bytes.
int check_tile_range(const std::vector<int> &ns, int L, int n_nu) {
    for (size_t a = 0; a < ns.size(); ++a) {
        const SlabTiles t = slab_tiles(ns[a], L, n_nu);
        if ((long long)t.nwb * t.bstride * 16 > 2147483647LL)
            return fail(RT_EINVAL, slab_name((long long)a) +
                                       ": the coefficient tiles of one direction exceed 2 GiB "
                                       "(too many frequencies for this depth grid)");
    }
    return RT_OK;
}

int plan_sweeps(rt_handle *h, const rt_problem *p, std::vector<double> &opac_c,
                std::vector<double> &wphi_c) {
    const rt_options &opt = h->opt;
    h->nc = merge_frequencies(p, opac_c, wphi_c);
    const int rays = h->M * h->nc;
    h->L = opt.chunk ? opt.chunk : auto_chunk(h->ns, rays);
    for (int n : h->ns)
        if ((long long)kWave * h->L < n - 1)
            return fail(RT_EINVAL, "options.chunk too short for ns (need 64 * chunk >= ns - 1)");
    // the same test as rt_validate, which does not look for equal opacities
    const int rc = check_tile_range(
        h->ns, opt.chunk ? opt.chunk : auto_chunk(h->ns, h->M * h->n_nu), h->n_nu);
    if (rc != RT_OK) return rc;
    // Waves per block, waves per direction and wave-batches per wave.
    //
    // Four waves per block; eight for a single slab, whose Arnoldi step adds up
    // the blocks' sums in one workgroup (200 points, 20 x 101 rays: GMRES 1.55
    // -> 1.51 ms, the operator alone the same), as long as their sums fit a row
    // each: eight waves that fill a shared row in turn take longer than four with
    // rows (512 points, 16 x 64 rays: operator 20.2 us against 11.8, GMRES 4.53
    // ms against 3.26).  Eight are compiled for chunks up to 8 only: longer ones
    // take four, also where the caller asked for eight and left the chunk to the
    // slabs' depths.
    const auto rows_fit = [&](int waves) {
        return (size_t)(waves + 1) * 2 * h->ns_max * sizeof(double) <= (size_t)kSweepLdsBudget;
    };
    h->W = opt.sweep_waves ? opt.sweep_waves : h->n_atm == 1 && rows_fit(8) ? 8 : 4;
    if (h->L > 8) h->W = 4;
    int wpd = h->W;
    bool whole = false;
    // One small slab: all of its directions in one block if that leaves a wave
    // at most four batches; the block then ends the operator itself and the
    // finalize launch goes (40 points, 8 x 21 rays: 9.8 -> 7.2 us back to back).
    {
        int w1 = h->W;
        while (w1 > 1 && (h->W / w1) < h->M) w1 /= 2;
        const int nwb = slab_tiles(h->ns[0], h->L, h->nc).nwb;
        if (opt.wave_batches == 0 && h->n_atm == 1 && h->L == 4 && h->W / w1 >= h->M &&
            (nwb + w1 - 1) / w1 <= 4 && rows_fit(h->W)) {
            wpd = w1;
            whole = true;
        }
    }
    // DELO-parabolic, whose bodies leave two waves per SIMD: four waves per block
    // for any other single slab (200 points, 20 x 101 rays: operator 11.0 -> 10.2
    // us, GMRES 759 -> 652 us; 400 points, 32 x 201: 13.8 -> 12.1, 2.05 -> 2.10 ms).
    if (!opt.sweep_waves && h->fs == RT_FS_DELO_PARABOLIC && !whole) h->W = wpd = 4;
    const long long dirs_total = (long long)h->n_atm * h->M;
    long long batches_total = 0;
    for (int n : h->ns) batches_total += (long long)h->M * slab_tiles(n, h->L, h->nc).nwb;
    // Big batches: the fewest waves per direction (a power of two) that still
    // give five waves per SIMD, so that what a wave does once -- sources,
    // depth steps, the sum over its rays -- is shared by more of its ray
    // batches.  FP64 / FP32 operator, slabs of 64 to 512 points, 16 directions,
    // 101 frequencies, us with 4, 2 and 1 waves per direction: 256 slabs
    // 65 / 35, 61 / 35, 85 / 50; 320 slabs 89 / 41, 85 / 39, 100 / 52; 512
    // slabs 136 / 66, 126 / 59, 124 / 69; 1024 slabs 263 / 140, 242 / 124,
    // 233 / 124.  Not where a block would then have places for twice the slab's
    // directions or more, and half of its waves nothing to do (6000 slabs of 64 to
    // 128 points, 2 directions of one |mu|, 51 frequencies: 57 us with four waves
    // on it, 77 with one and three idle).
    if (opt.wave_batches == 0 && !whole)
        while (wpd > 1 && dirs_total * (wpd / 2) >= 5 * 4 * 256 && h->W / (wpd / 2) < 2 * h->M)
            wpd /= 2;
    // FP32 sweeps: no wave adds up more ray batches in FP32 than it would with a
    // ray per frequency and every wave of a block on one direction (512 and 1024
    // slabs of distinct opacities, errors against the FP64 operator 2.04e-7 and
    // 1.51e-7 normwise with the waves per direction above, 1.93e-7 and 1.34e-7 so).
    int wpd32 = wpd;
    for (int n : h->ns) {
        const int now = slab_tiles(n, h->L, h->nc).nwb, all = slab_tiles(n, h->L, h->n_nu).nwb;
        while (!whole && wpd32 < h->W && (now + wpd32 - 1) / wpd32 > (all + h->W - 1) / h->W) wpd32 *= 2;
    }
    // Small ones: several blocks per direction, two waves per SIMD in all but
    // at least two batches per wave (below that a block's fixed part costs
    // more than the shorter chain saves).  With about 48 blocks in all
    // instead: one 1024-point slab 30.8 -> 24.6 us FP64, 21.6 -> 16.1 FP32; 8
    // slabs 16.7 -> 10.4; 32 slabs 22.9 -> 17.7; 64 slabs 24.8 -> 23.0.  Bodies of
    // chunks longer than 8 leave one FP64 wave per SIMD, so there one wave per SIMD
    // in all, if the directions leave room for it: a second round of blocks of two
    // batches takes as long as the first.  FP64 operator with two and one, us: one
    // 1024-point slab of 32 x 201 distinct rays 42.6 and 28.0, 3 slabs of 1000
    // points and 16 x 101 41.5 and 25.9, 8 slabs of 1024 points 48.8 and 34.6;
    // but 40 slabs of 700, whose 320 directions do not fit one round, 58.7 and 67.8.
    const long long fill_waves = (h->L > 8 && dirs_total <= 256 ? 1 : 2) * 4 * 256;
    const int nb_fill = (int)std::max<long long>(2, (batches_total + fill_waves - 1) / fill_waves);
    // The plan that the Arnoldi step reads: at least kSolveWb batches per wave,
    // but two where a single slab then has no more than kOneXcd blocks.
    const int slab_blocks = h->M * ((slab_tiles(h->ns_max, h->L, h->nc).nwb + 2 * h->W - 1) / (2 * h->W));
    const int solve_wb = h->n_atm == 1 && slab_blocks <= kOneXcd ? 2 : kSolveWb;
    std::vector<AtmDesc> atm(h->n_atm);
    std::vector<int> nb(h->n_atm), nb32(h->n_atm), nb_tail(h->n_atm);
    for (int a = 0; a < h->n_atm; ++a) {
        AtmDesc &d = atm[a];
        d.ns = h->ns[a];
        d.doff = h->doff[a];
        const SlabTiles t = slab_tiles(d.ns, h->L, h->nc);
        d.C = t.C;
        d.Leff = t.Leff;
        d.nlong = t.nlong;
        d.G = t.G;
        d.n_nu = h->nc;
        d.nwb = t.nwb;
        d.bstride = t.bstride;
        d.ray_off = a * rays;
        d.coef_off = h->n_pairs;
        d.q_off = h->n_qt;
        d.a_off = h->n_dense;
        d.ew_off = h->n_ew;
        h->n_pairs += (long long)h->M * d.nwb * d.bstride;
        h->n_qt += (long long)h->M * d.nwb * d.G;
        h->n_dense += 4LL * d.ns * d.ns;
        h->n_ew += (long long)(d.ns - 1) * rays;
        d.eps = p->eps[a];
        d.xi = 1.0 - p->eps[a];
        d.W2 = p->W2[a];
        d.Ibot = p->I_bot ? p->I_bot[a] : (p->B ? p->B[d.doff + d.ns - 1] : 1.0);
        nb[a] = std::min(std::min(nb_fill, 32), (d.nwb + wpd - 1) / wpd);
        if (wpd < h->W || whole) nb[a] = (d.nwb + wpd - 1) / wpd;
        if (opt.wave_batches > 0) nb[a] = opt.wave_batches;
        nb32[a] = std::min((d.nwb + wpd32 - 1) / wpd32, 32);
        // a plan the caller fixed is kept for every cycle
        nb_tail[a] = opt.wave_batches > 0 ? nb[a] : std::min(std::max(nb[a], solve_wb), kTailWb);
    }
    h->main = make_plan(atm, h->M, h->W, wpd, nb);
    h->main.whole = whole;
    if (wpd32 != wpd && sweeps_fp32(h, true)) h->main32 = make_plan(atm, h->M, h->W, wpd32, nb32);
    // the tail plan, over the same tiles, only where it differs
    SweepPlan tail = make_plan(atm, h->M, h->W, h->W, nb_tail);
    if (tail.n_blocks != h->main.n_blocks) h->tail = std::move(tail);
    // A single slab of few blocks: all of them on one XCD (workgroups go to
    // the 8 in turn: every eighth place of the grid, the others empty), so that
    // the workgroup that reads their sums, the first of its grid, finds them in
    // its L2: 200 points, 20 x 101 rays, 40 blocks of 8 waves, 20.9 -> 19.8 us a
    // GMRES step.  More blocks take turns on its 32 CUs: 64 of 8 waves (400
    // points, 32 x 201 rays) 26.5 us on all XCDs, 34.8 on one; 56 (283 points, 16 x
    // 101 distinct rays) 23.1 and 25.8, or 22.1 as 32 blocks of four batches per
    // wave on one.  The operator alone ends in a pass over all XCDs and keeps them.
    SweepPlan &solve = h->tail.n_blocks ? h->tail : h->main;
    if (h->n_atm == 1 && solve.n_blocks > 1 && solve.n_blocks <= kOneXcd && h->ns_max <= 512)
        solve.spread = 3;
    h->n_partial = std::max({h->main.n_partial, h->main32.n_partial, h->tail.n_partial});
    return RT_OK;
}

}  // namespace rt
