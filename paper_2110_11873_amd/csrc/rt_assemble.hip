// rt_assemble.hip -- dense assembly of A = Id - J Lambda T on gfx950.
//
// Sect. 3.3 assembles A column by column, applying Algorithm 1 to the unit
// vectors; a point source at depth j leaves the intensity zero upwind of j
// and only decays downwind of it (Sect. 4.4).  Here the columns of a block of
// 64 source depths are built together by a multi-source sweep in tiles of 16
// depths:
//
//  * a wavefront owns one |mu| and up to RG frequencies of it; its lanes hold,
//    for 16 columns and four groups of rays, the intensities I_r(b; j) at the
//    first depth b of a tile, pre-multiplied by the ray weight q_r;
//  * downwind of the sources row k of a tile is sum_r X_r(k) I_r(b; j), X_r(k)
//    the product of the rays' E from b to k: a 16 x RG by RG x 16 product on
//    the FP64 matrix cores (the intensities are their B operand as they stand,
//    X comes from a table in the A operand's order), one multiply-add per
//    (depth, column, ray) where stepping the rays one depth at a time takes a
//    multiply, an add and a coefficient from LDS.  Then I(b) *= the tile's
//    transmission, and the next tile follows;
//  * in the tile that holds the columns' own depths the rays are stepped: the
//    intensity starts at k = j (through c_k of the interval entering j), picks
//    up the source at k = j + 1 (through c_u), then only decays;
//  * the T^2_0 weights of the wavefront's |mu| turn its rows into the three
//    moments sum q Lambda, sum q T1 Lambda, sum q (T1^2 + T2^2) Lambda that
//    make up the 2x2 block of A at (k, j) (eqs. J00/J02 with S_I = s00 + T1
//    s20, S_Q = T2 s20), added over the wavefronts of a workgroup through LDS
//    in a fixed order once per tile.
//
// The downward rays give the lower triangle (k > j), the upward rays -- the
// same code on the reversed depth order -- the upper one; the 2x2 blocks on
// the diagonal receive both and are written by a separate pass.  When a
// workgroup cannot hold every ray, the rays are split into slices whose
// moments are stored apart and added, in slice order, by a combine pass.
// Nothing is accumulated with atomics: the result is bitwise reproducible.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>
#include <vector>

#include "rt_coef.h"
#include "rt_internal.h"

namespace rt {

namespace {

struct AsmTask {
    int atm;    // slab
    int dir;    // 0: mu < 0 (downward, lower triangle), 1: mu > 0 (upward, upper)
    int jblk;   // block of 64 source depths, in the direction's depth order
    int slice;  // ray slice
};

struct AsmArgs {
    const AtmDesc *atm;
    const AsmTask *task;
    const double2 *ew;       // (E, w) per slab, interval and ray
    const double *xt, *tt;   // tile transmissions: tile_table_kernel
    const long long *tile0;  // per slab: tiles of the slabs before it in its group
    int slab0;               // tile_table_kernel: the group's first slab
    const RayConst *rayc;
    const double2 *dirc;     // per |mu|: (T1, T1^2 + T2^2)
    double *A;               // final A, or the raw moments of slice 0
    double *sc;              // raw moments of slices 1.. (stride sc_stride)
    long long sc_stride;
    double *dg;              // [slice][dir][ns_total][3] moments of the diagonal blocks
    int ns_total;
    int n_nu, M;
    int rg;                  // ray slots per wavefront
    int cpm;                 // wavefronts (frequency groups) per |mu|
    int nw;                  // wavefronts per workgroup
    int slices;
};

// (E, w) per (slab, interval i = 1..ns-1 between depths i-1 and i, ray
// r = m n_nu + p), at ew_off + (i - 1) (M n_nu) + r.
__global__ void ew_table_kernel(const AtmDesc *atm, const double *tau, const double *opac,
                                const double *mu_pos, int M, int n_nu, int fs, double2 *ew) {
    const AtmDesc at = atm[blockIdx.y];
    const int R = M * n_nu;
    const long long n = (long long)(at.ns - 1) * R;
    for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < n;
         e += (long long)gridDim.x * blockDim.x) {
        const int i = (int)(e / R) + 1, r = (int)(e % R);
        const int m = r / n_nu, p = r % n_nu;
        const double kap = opac[(long long)blockIdx.y * n_nu + p] / mu_pos[m];
        const double d = kap * (tau[at.doff + i] - tau[at.doff + i - 1]);
        double E, w;
        step_ew(fs, d, E, w);
        ew[at.ew_off + e] = make_double2(E, w);
    }
}

constexpr int kTile = 16;                    // depths per tile: rows of an MFMA
constexpr int kAsmNT = 512;                  // threads of the largest workgroup
constexpr int kRedRow = kWave + 8;           // padded row of the wavefronts' sums in LDS
constexpr int kRed = kTile * kRedRow;        // one wavefront's 16 x 64 sums
typedef double v4d __attribute__((ext_vector_type(4)));

// E entering depth k of the direction's order (k = 1 .. ns - 1), 1 elsewhere;
// the interval's row in the (E, w) table.
__device__ inline int ew_row(int dir, int k, int ns) { return dir == 0 ? k - 1 : ns - 1 - k; }

// Products of E within the tiles of 16 depths (in the direction's order), per
// wavefront chunk c and ray slot.  With b the tile's first depth:
//   xt[((tile nchunks + c) RG + slot) 16 + row] = E_{b+1} .. E_{b+row}
//   tt[ (tile nchunks + c) RG + slot]           = E_{b+1} .. E_{b+16}
// tile = 2 tile0 + dir ntiles + b / 16.  Slot 4 i + g holds ray g RG/4 + i of
// the chunk, so a wavefront reads step i of its A operand -- 16 rows of the
// four rays that its four lane groups hold -- as 64 consecutive entries.
__global__ void tile_table_kernel(AsmArgs g, double *xt, double *tt) {
    const int slab = g.slab0 + blockIdx.y;
    const AtmDesc at = g.atm[slab];
    const int ns = at.ns, nt = (ns + kTile - 1) / kTile;
    if ((int)blockIdx.x >= 2 * nt) return;
    const int dir = blockIdx.x / nt, b = (blockIdx.x % nt) * kTile;
    const int nchunks = g.M * g.cpm, R = g.M * g.n_nu, RI = g.rg / 4;
    const long long tile = 2 * g.tile0[slab] + blockIdx.x;
    // the products of 256 rays at a time in LDS (rays in the order of the (E, w)
    // table, then slots in the order of the output)
    __shared__ double Xs[256 * (kTile + 1)];
    for (int s0 = 0; s0 < nchunks * g.rg; s0 += 256) {
        const int s = s0 + threadIdx.x, c = s / g.rg, rr = s % g.rg, p = (c % g.cpm) * g.rg + rr;
        __syncthreads();
        if (c < nchunks) {
            const double2 *ew = g.ew + at.ew_off + (c / g.cpm) * g.n_nu + p;
            double E[kTile], X = 1.0;
#pragma unroll
            for (int i = 0; i < kTile; ++i) {
                const int k = b + 1 + i;
                E[i] = p < g.n_nu && k < ns ? ew[(long long)ew_row(dir, k, ns) * R].x : 1.0;
            }
#pragma unroll
            for (int i = 0; i < kTile; ++i) {
                Xs[threadIdx.x * (kTile + 1) + i] = X;
                X *= E[i];
            }
            tt[tile * nchunks * g.rg + (long long)c * g.rg + 4 * (rr % RI) + rr / RI] = X;
        }
        __syncthreads();
        for (int e = threadIdx.x; e < 256 * kTile; e += 256) {
            const int x = e / kTile, row = e % kTile, sx = s0 + x, cx = sx / g.rg, rx = sx % g.rg;
            if (cx < nchunks)
                xt[(tile * nchunks * g.rg + (long long)cx * g.rg + 4 * (rx % RI) + rx / RI) * kTile + row] =
                    Xs[x * (kTile + 1) + row];
        }
    }
}

// LDS before the ray weights, in doubles: two tiles' sums, or the staged (E, w).
__host__ __device__ constexpr int asm_lds_head(int nw, int rg) {
    const int sums = 2 * nw * kRed, staged = 2 * nw * (kTile + 1) * rg;
    return sums > staged ? sums : staged;
}

// One workgroup per task, a wavefront per chunk of at most RG rays.  LDS: the
// wavefronts' sums of two tiles; in the tiles that hold the task's columns,
// in their place, the (E, w) of the wavefronts' rays for 17 depths; then the
// ray weights and the wavefronts' T^2_0 weights.  Operand layout of v_mfma_f64_16x16x4: lane l feeds
// A[l % 16][l / 16] and B[l / 16][l % 16], result register r of lane l is
// D[4 r + l / 16][l % 16].  Held to two waves per SIMD by the intensities of
// 64 columns (2 RG registers), so what bounds it is latency at one workgroup
// per CU: 512 slabs of 64 to 512 points, 8 |mu| x 51 opacities, take 1.97 ms
// (5.11 ms stepping every depth); without its own tiles it would take 1.37,
// without the sums and the stores of 1.7 GB 1.72, without the products 1.90.
template <int RG>
__global__ __launch_bounds__(kAsmNT)
__attribute__((amdgpu_waves_per_eu(2, 2))) void assemble_kernel(AsmArgs g) {
    static_assert(RG % 4 == 0 && RG <= kWave, "four lane groups; one staged ray per lane");
    constexpr int RI = RG / 4, CT = kWave / kTile;
    extern __shared__ double smem[];
    const AsmTask t = g.task[blockIdx.x];
    const AtmDesc at = g.atm[t.atm];
    const int ns = at.ns, R = g.M * g.n_nu, nw = g.nw;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = threadIdx.x % kWave, col = lane % kTile, sub = lane / kTile;
    const int nt = (ns + kTile - 1) / kTile;
    const int nchunks = g.M * g.cpm;
    const int c = t.slice * nw + wave, cc = min(c, nchunks - 1);
    const int p0 = (cc % g.cpm) * RG, m = cc / g.cpm;

    double *red = smem;                                           // [2][nw][kRed]
    double2 *ew_s = reinterpret_cast<double2 *>(smem) + wave * (kTile + 1) * RG;
    double *q_s = smem + asm_lds_head(nw, RG) + wave * RG;
    const bool my_ray = c < nchunks && lane < RG && p0 + lane < g.n_nu;
    const int my_r = m * g.n_nu + (my_ray ? p0 + lane : 0);
    if (lane < RG) q_s[lane] = my_ray ? g.rayc[at.ray_off + my_r].q : 0.0;
    double2 *tw_s = reinterpret_cast<double2 *>(smem + asm_lds_head(nw, RG) + nw * RG);
    if (lane == 0) tw_s[wave] = g.dirc[m];  // (T1, T1^2 + T2^2)

    // ray sub RI + i of the chunk, at the first depth of the tile, for the
    // columns 16 ct + col of the block
    double It[CT][RI];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int i = 0; i < RI; ++i) It[ct][i] = 0.0;

    const int j0 = t.jblk * kWave, kt0 = j0 / kTile;  // the block's first tile
    const long long tile0 = 2 * g.tile0[t.atm] + (long long)t.dir * nt;

    // the tile at depths b .. b + 15, whose columns are the tile's own: cur
    // <- the intensities at b + 16, acc <- the rows in the products' layout
    auto own_tile = [&](int b, double (&cur)[RI], v4d &acc) {
        // (loads without a branch, nine in flight: one at a time, waiting for
        // each, they took 1 ms of 2.4 for 512 slabs)
        const double2 *from = g.ew + at.ew_off + my_r;
        constexpr int kHalf = kTile / 2 + 1;
#pragma unroll
        for (int h = 0; h <= kTile; h += kHalf) {
            double2 v[kHalf];
#pragma unroll
            for (int u = 0; u < kHalf; ++u) {
                const int k = max(1, min(b + h + u, ns - 1));
                v[u] = from[(long long)ew_row(t.dir, k, ns) * R];
            }
#pragma unroll
            for (int u = 0; u < kHalf; ++u) {
                const int k = b + h + u;
                const bool on = my_ray && k >= 1 && k < ns;
                v[u].x = on ? v[u].x : 1.0;
                v[u].y = on ? v[u].y : 1.0;
            }
            if (lane < RG) {
#pragma unroll
                for (int u = 0; u < kHalf; ++u)
                    if (h + u <= kTile) ew_s[(h + u) * RG + lane] = v[u];
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");  // this wavefront's own rows
        __builtin_amdgcn_wave_barrier();
        // the sources: q c_k at k = j, and that carried to k = j + 1 with q c_u
        double s1[RI], first = 0.0;
#pragma unroll
        for (int i = 0; i < RI; ++i) {
            const int rr = sub * RI + i;
            const double2 e0 = ew_s[col * RG + rr], e1 = ew_s[(col + 1) * RG + rr];
            const double q = q_s[rr], ck = q * (1.0 - e0.y);
            first += ck;
            s1[i] = fma(e1.x, ck, q * (e1.y - e1.x));
            cur[i] = 0.0;
        }
        auto advance = [&](int st) {
            // (zero above the source; 0/1 factor: a select would load E in a branch)
            const double2 *row = ew_s + st * RG + sub * RI;
            const double f = col == st - 1 ? 1.0 : 0.0;
#pragma unroll
            for (int i = 0; i < RI; ++i) cur[i] = fma(f, s1[i], cur[i] * row[i].x);
        };
        // four depths at a time, their sums over the lane groups exchanged
        // together: group u ends with depth 4 r + u.  Rolled, and the depths
        // kept apart: reads hoisted from later ones spill the intensities
#pragma unroll 1
        for (int r = 0; r < 4; ++r) {
            double a[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int st = 4 * r + u;
                if (st > 0) advance(st);
                double a0 = col == st ? first : 0.0, a1 = 0.0;
#pragma unroll
                for (int i = 0; i < RI; ++i) {
                    if (i & 1) a1 += cur[i];
                    else a0 += cur[i];
                }
                a[u] = a0 + a1;
                __builtin_amdgcn_sched_barrier(0);
            }
            const bool hi = sub & 2, odd = sub & 1;
            const double b0 = (hi ? a[2] : a[0]) + __shfl_xor(hi ? a[0] : a[2], 32);
            const double b1 = (hi ? a[3] : a[1]) + __shfl_xor(hi ? a[1] : a[3], 32);
            const double sum = (odd ? b1 : b0) + __shfl_xor(odd ? b0 : b1, 16);
#pragma unroll
            for (int u = 0; u < 4; ++u) acc[u] = r == u ? sum : acc[u];
        }
        advance(kTile);
    };

    // the wavefront's rows into LDS
    auto put_sums = [&](int buf, const v4d (&acc)[CT]) {
        double *mine = red + (buf * nw + wave) * kRed;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int r = 0; r < 4; ++r) mine[(4 * r + sub) * kRedRow + kTile * ct + col] = acc[ct][r];
    };
    // add the wavefronts' rows of tile kt with their weights and write A
    auto finish = [&](int kt, int buf) {
        for (int e = threadIdx.x; e < kTile * kWave; e += blockDim.x) {
            const int row = e / kWave, l = e % kWave;
            const int k = kt * kTile + row, j = j0 + l;
            if (k >= ns || j > k) continue;
            double v0 = 0.0, v1 = 0.0, v2 = 0.0;
#pragma unroll 4
            for (int w = 0; w < nw; ++w) {
                const double x = red[(buf * nw + w) * kRed + row * kRedRow + l];
                const double2 tw = tw_s[w];
                v0 += x;
                v1 = fma(tw.x, x, v1);
                v2 = fma(tw.y, x, v2);
            }
            const int K = t.dir == 0 ? k : ns - 1 - k, J = t.dir == 0 ? j : ns - 1 - j;
            if (K == J) {
                double *d = g.dg + (((long long)t.slice * 2 + t.dir) * g.ns_total + at.doff + K) * 3;
                d[0] = v0;
                d[1] = v1;
                d[2] = v2;
                continue;
            }
            const long long N = 2LL * ns, base = at.a_off + 2LL * K * N + 2LL * J;
            if (g.slices == 1) {
                *reinterpret_cast<double2 *>(g.A + base) = make_double2(-at.xi * v0, -at.xi * v1);
                *reinterpret_cast<double2 *>(g.A + base + N) =
                    make_double2(-at.xi * at.W2 * v1, -at.xi * at.W2 * v2);
            } else {
                double *out = t.slice == 0 ? g.A : g.sc + (t.slice - 1) * g.sc_stride;
                *reinterpret_cast<double2 *>(out + base) = make_double2(v0, v1);
                out[base + N + 1] = v2;
            }
        }
    };

    // a tile's A operands and the lane's rays' transmissions across it
    auto load_x = [&](int kt, double (&x)[RI]) {
        const double *from = g.xt + ((tile0 + min(kt, nt - 1)) * nchunks + cc) * RG * kTile + lane;
#pragma unroll
        for (int i = 0; i < RI; ++i) x[i] = from[i * kWave];
    };
    auto load_t = [&](int kt, double (&tr)[RI]) {
        const double *from = g.tt + ((tile0 + kt) * nchunks + cc) * RG + sub;
#pragma unroll
        for (int i = 0; i < RI; ++i) tr[i] = from[4 * i];
    };

    // the block's own tiles: columns of the tiles before by the product, the
    // tile's own stepped, later columns not reached yet
#pragma unroll
    for (int t4 = 0; t4 < CT; ++t4) {
        const int kt = kt0 + t4;
        if (kt >= nt) continue;
        v4d acc[CT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[ct] = v4d{0.0, 0.0, 0.0, 0.0};
        if (t4 > 0) {
            double x[RI], tr[RI];
            load_x(kt, x);
            load_t(kt, tr);
#pragma unroll
            for (int i = 0; i < RI; ++i)
#pragma unroll
                for (int ct = 0; ct < t4; ++ct)
                    acc[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[i], It[ct][i], acc[ct], 0, 0, 0);
#pragma unroll
            for (int i = 0; i < RI; ++i)
#pragma unroll
                for (int ct = 0; ct < t4; ++ct) It[ct][i] *= tr[i];
        }
        __syncthreads();  // the sums of the tile before are read: their place is free
        own_tile(kt * kTile, It[t4], acc[t4]);
        __syncthreads();  // every wavefront has read its staged coefficients
        put_sums(0, acc);
        __syncthreads();
        finish(kt, 0);
    }
    // the tiles below, the next one's operands loaded during the products.
    // (One of a SIMD's two wavefronts adding up a tile while the other's
    // products run measured no better: 2.51 ms against 2.39 for 512 slabs.)
    double x[RI];
    load_x(kt0 + CT, x);
    for (int kt = kt0 + CT; kt < nt; ++kt) {
        v4d acc[CT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[ct] = v4d{0.0, 0.0, 0.0, 0.0};
        double xn[RI], tr[RI];
        load_t(kt, tr);
        load_x(kt + 1, xn);
#pragma unroll
        for (int i = 0; i < RI; ++i)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
                acc[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[i], It[ct][i], acc[ct], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < RI; ++i) {
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) It[ct][i] *= tr[i];
            x[i] = xn[i];
        }
        const int buf = (kt - kt0 - CT + 1) & 1;
        put_sums(buf, acc);
        __syncthreads();
        finish(kt, buf);
    }
}

// Off-diagonal 2x2 blocks from the slices' raw moments (slices > 1).
__global__ void assemble_combine_kernel(AsmArgs g) {
    const AtmDesc at = g.atm[blockIdx.y];
    const long long ns = at.ns, N = 2 * ns;
    for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < ns * ns;
         e += (long long)gridDim.x * blockDim.x) {
        const long long K = e / ns, J = e % ns;
        if (K == J) continue;
        const long long base = at.a_off + 2 * K * N + 2 * J;
        double v0 = g.A[base], v1 = g.A[base + 1], v2 = g.A[base + N + 1];
        for (int s = 1; s < g.slices; ++s) {
            const double *b = g.sc + (s - 1) * g.sc_stride;
            v0 += b[base];
            v1 += b[base + 1];
            v2 += b[base + N + 1];
        }
        g.A[base] = -at.xi * v0;
        g.A[base + 1] = -at.xi * v1;
        g.A[base + N] = -at.xi * at.W2 * v1;
        g.A[base + N + 1] = -at.xi * at.W2 * v2;
    }
}

// The 2x2 blocks on the diagonal: both directions, all slices, plus Id.
__global__ void assemble_diag_kernel(AsmArgs g, const int *pt_atm) {
    const int kk = blockIdx.x * blockDim.x + threadIdx.x;
    if (kk >= g.ns_total) return;
    const AtmDesc at = g.atm[pt_atm[kk]];
    const long long K = kk - at.doff, N = 2LL * at.ns;
    double v[3] = {0.0, 0.0, 0.0};
    for (int s = 0; s < g.slices; ++s)
        for (int d = 0; d < 2; ++d)
            for (int mom = 0; mom < 3; ++mom)
                v[mom] += g.dg[(((long long)s * 2 + d) * g.ns_total + kk) * 3 + mom];
    double *A = g.A + at.a_off + 2 * K * N + 2 * K;
    A[0] = 1.0 - at.xi * v[0];
    A[1] = -at.xi * v[1];
    A[N] = -at.xi * at.W2 * v[1];
    A[N + 1] = 1.0 - at.xi * at.W2 * v[2];
}

// Compiled variants: ray slots per wavefront, at most 8 wavefronts per
// workgroup.  52 slots are the most whose intensities, operands and sums fit
// 256 registers with the next tile's operands in flight.
constexpr int kVariants[] = {8, 16, 28, 40, 52};
constexpr int kAsmWaves = kAsmNT / kWave;

template <int RG>
hipError_t launch_variant(const AsmArgs &a, int ntasks, hipStream_t s) {
    const size_t lds = (asm_lds_head(a.nw, RG) + (size_t)a.nw * (RG + 2)) * sizeof(double);
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void *)assemble_kernel<RG>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((assemble_kernel<RG>), dim3(ntasks), dim3(kWave * a.nw), lds, s, a);
    return hipGetLastError();
}

hipError_t launch_assemble(const AsmArgs &a, int ntasks, hipStream_t s) {
    switch (a.rg) {
        case 8: return launch_variant<8>(a, ntasks, s);
        case 16: return launch_variant<16>(a, ntasks, s);
        case 28: return launch_variant<28>(a, ntasks, s);
        case 40: return launch_variant<40>(a, ntasks, s);
        default: return launch_variant<52>(a, ntasks, s);
    }
}

template <typename T>
int alloc(T **p, size_t count) {
    if (count == 0) count = 1;
    if (hipMalloc((void **)p, count * sizeof(T)) != hipSuccess) {
        *p = nullptr;
        (void)hipGetLastError();
        return fail(RT_ENOMEM, "device allocation of " + std::to_string(count * sizeof(T)) +
                                   " bytes for the dense assembly failed");
    }
    return RT_OK;
}

AsmArgs asm_args(const rt_handle *h) {
    AsmArgs g{};
    g.atm = h->d_atm;
    g.task = static_cast<const AsmTask *>(h->d_asm_task);
    g.ew = h->d_ew;
    g.xt = h->d_asm_xt;
    g.tt = h->d_asm_tt;
    g.tile0 = h->d_asm_tile0;
    g.rayc = h->d_rayc;
    g.dirc = h->d_dirc;
    g.sc = h->d_asm_sc;
    g.sc_stride = h->n_dense;
    g.dg = h->d_asm_dg;
    g.ns_total = h->ns_total;
    g.n_nu = h->nc;
    g.M = h->M;
    g.rg = h->asm_rg;
    g.cpm = h->asm_cpm;
    g.nw = h->asm_nw;
    g.slices = h->asm_slices;
    return g;
}

// The tile transmissions of one group of slabs.
int fill_tables(const rt_handle *h, const rt_handle::AsmGroup &gr, hipStream_t s) {
    AsmArgs g = asm_args(h);
    g.slab0 = gr.slab0;
    int ns_max = 1;
    for (int a = gr.slab0; a < gr.slab1; ++a) ns_max = std::max(ns_max, h->ns[a]);
    hipLaunchKernelGGL(tile_table_kernel, dim3(2 * ((ns_max + kTile - 1) / kTile), gr.slab1 - gr.slab0),
                       dim3(256), 0, s, g, h->d_asm_xt, h->d_asm_tt);
    if (hipGetLastError() != hipSuccess) return fail(RT_EDEVICE, "assembly tile table launch failed");
    return RT_OK;
}

// Plan the assembly once per handle: frequency groups of RG rays per
// wavefront (the fewest slices, then the smallest RG), wavefronts per
// workgroup, the task list (longest walks first) and the workspace.
//
// The tile transmissions take as much memory again as the (E, w) table (17 bytes
// per depth and ray slot; 512 slabs of 64 to 512 points, 8 |mu| x 51 distinct
// opacities: 1.1 GB, kept on the handle).  Where there is no room for all of them, the
// slabs are assembled in groups that share the memory of the largest group, whose
// tables are then made in every call.
int plan_assembly(rt_handle *h, hipStream_t s) {
    if (h->d_asm_task) return RT_OK;
    // the fewest slices, then the fewest empty ray slots, then the smaller variant
    int best_rg = 0, best_slices = 0, best_nw = 0;
    long long best_waste = 0;
    for (const int rg : kVariants) {
        const int cpm = (h->nc + rg - 1) / rg;
        const int chunks = h->M * cpm;
        const int slices = (chunks + kAsmWaves - 1) / kAsmWaves;
        const int nw = (chunks + slices - 1) / slices;
        const long long waste = (long long)slices * nw * rg - (long long)h->M * h->nc;
        if (!best_rg || slices < best_slices || (slices == best_slices && waste < best_waste)) {
            best_rg = rg;
            best_slices = slices;
            best_nw = nw;
            best_waste = waste;
        }
    }
    h->asm_rg = best_rg;
    h->asm_cpm = (h->nc + best_rg - 1) / best_rg;
    h->asm_slices = best_slices;
    h->asm_nw = best_nw;
    // groups of consecutive slabs of about tiles / n tiles each
    long long tiles = 0;
    for (int n : h->ns) tiles += (n + kTile - 1) / kTile;
    std::vector<long long> tile0(h->n_atm);
    std::vector<AsmTask> tasks;
    long long most = 0;  // tiles of the largest group
    auto split = [&](int n) {
        h->asm_groups.clear();
        tasks.clear();
        most = 0;
        for (int a = 0; a < h->n_atm;) {
            rt_handle::AsmGroup gr{a, a, (int)tasks.size(), 0};
            long long t = 0;
            for (; gr.slab1 < h->n_atm && (t == 0 || t < (tiles + n - 1) / n); ++gr.slab1) {
                tile0[gr.slab1] = t;
                t += (h->ns[gr.slab1] + kTile - 1) / kTile;
            }
            for (; a < gr.slab1; ++a)
                for (int d = 0; d < 2; ++d)
                    for (int jb = 0; jb * kWave < h->ns[a]; ++jb)
                        for (int sl = 0; sl < best_slices; ++sl) tasks.push_back(AsmTask{a, d, jb, sl});
            gr.tasks = (int)tasks.size() - gr.task0;
            // longest walks first.  (A slab's tasks, which read the same tile table, on
            // one XCD measured 2.50 ms against 2.39 for 512 slabs.)
            std::stable_sort(tasks.begin() + gr.task0, tasks.end(),
                             [&](const AsmTask &x, const AsmTask &y) {
                                 return h->ns[x.atm] - kWave * x.jblk > h->ns[y.atm] - kWave * y.jblk;
                             });
            most = std::max(most, t);
            h->asm_groups.push_back(gr);
        }
    };
    int rc;
    // the task list is set on the handle last, after the tables' launches: it
    // marks the plan as made, so a failure frees whatever this call allocated and
    // a later call starts over
    AsmTask *dt = nullptr;
    auto undo = [&](int code) {
        for (void **q : {(void **)&dt, (void **)&h->d_ew, (void **)&h->d_asm_dg,
                         (void **)&h->d_asm_sc, (void **)&h->d_asm_xt, (void **)&h->d_asm_tt,
                         (void **)&h->d_asm_tile0}) {
            if (*q) (void)hipFree(*q);
            *q = nullptr;
        }
        return code;
    };
    if ((rc = alloc(&h->d_ew, (size_t)h->n_ew)) != RT_OK) return undo(rc);
    if ((rc = alloc(&h->d_asm_dg, (size_t)best_slices * 2 * h->ns_total * 3)) != RT_OK)
        return undo(rc);
    if (best_slices > 1 &&
        (rc = alloc(&h->d_asm_sc, (size_t)(best_slices - 1) * h->n_dense)) != RT_OK)
        return undo(rc);
    split(1);
    if ((rc = alloc(&dt, tasks.size())) != RT_OK) return undo(rc);
    if ((rc = alloc(&h->d_asm_tile0, tile0.size())) != RT_OK) return undo(rc);
    // the tile transmissions, of as few groups as there is room for
    for (int n = 2;; n *= 2) {
        const size_t slots = (size_t)2 * most * h->M * h->asm_cpm * best_rg;
        if ((rc = alloc(&h->d_asm_xt, slots * kTile)) == RT_OK &&
            (rc = alloc(&h->d_asm_tt, slots)) == RT_OK)
            break;
        if (h->d_asm_xt) (void)hipFree(h->d_asm_xt);
        h->d_asm_xt = nullptr;
        if ((int)h->asm_groups.size() == h->n_atm) return undo(rc);
        split(n);
    }
    if (hipMemcpy(dt, tasks.data(), tasks.size() * sizeof(AsmTask), hipMemcpyHostToDevice) !=
        hipSuccess)
        return undo(fail(RT_EDEVICE, "assembly task upload failed"));
    if (hipMemcpy(h->d_asm_tile0, tile0.data(), tile0.size() * sizeof(long long),
                  hipMemcpyHostToDevice) != hipSuccess)
        return undo(fail(RT_EDEVICE, "assembly tile table upload failed"));
    int ns_max_m1 = 1;
    for (int n : h->ns) ns_max_m1 = std::max(ns_max_m1, n - 1);
    const long long per = (long long)ns_max_m1 * h->M * h->nc;
    const dim3 grid((unsigned)std::min<long long>((per + 255) / 256, 4096), h->n_atm);
    hipLaunchKernelGGL(ew_table_kernel, grid, dim3(256), 0, s, h->d_atm, h->d_tau, h->d_opac_c,
                       h->d_mu_pos, h->M, h->nc, h->fs, h->d_ew);
    if (hipGetLastError() != hipSuccess)
        return undo(fail(RT_EDEVICE, "assembly coefficient launch failed"));
    if (h->asm_groups.size() == 1 && (rc = fill_tables(h, h->asm_groups[0], s)) != RT_OK)
        return undo(rc);
    h->d_asm_task = dt;
    return RT_OK;
}

}  // namespace

int assemble(rt_handle *h, double *A, hipStream_t s) {
    int rc = plan_assembly(h, s);
    if (rc != RT_OK) return rc;
    AsmArgs g = asm_args(h);
    g.A = A;
    const AsmTask *tasks = g.task;
    for (const rt_handle::AsmGroup &gr : h->asm_groups) {
        if (h->asm_groups.size() > 1 && (rc = fill_tables(h, gr, s)) != RT_OK) return rc;
        g.task = tasks + gr.task0;
        if (launch_assemble(g, gr.tasks, s) != hipSuccess)
            return fail(RT_EDEVICE, "assembly launch failed");
    }
    if (g.slices > 1) {
        long long nsq = 1;
        for (int n : h->ns) nsq = std::max(nsq, (long long)n * n);
        const dim3 grid((unsigned)std::min<long long>((nsq + 255) / 256, 4096), h->n_atm);
        hipLaunchKernelGGL(assemble_combine_kernel, grid, dim3(256), 0, s, g);
        if (hipGetLastError() != hipSuccess) return fail(RT_EDEVICE, "assembly combine launch failed");
    }
    hipLaunchKernelGGL(assemble_diag_kernel, dim3((h->ns_total + 255) / 256), dim3(256), 0, s, g,
                       (const int *)h->d_pt_atm);
    if (hipGetLastError() != hipSuccess) return fail(RT_EDEVICE, "assembly diagonal launch failed");
    return RT_OK;
}

}  // namespace rt
