// Born forward operator (paper, Inverse Problem section, Eqs. 8-9;
// linearisation of Eq. 1 in q = 1/c^2 with Green's functions from Eqs. 4-5).
//
//   d_er = omega^2 h^2 sum_x G_e(x) G_r(x) delta(x)
//
// A split-K complex GEMM over pixels on the matrix cores.  The output is
// symmetric in (e, r), so only upper-triangular tiles are computed; the
// split partials are reduced in a fixed order.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "born.h"
#include "common.h"
#include "mma.h"

namespace rb {
namespace {

// ------------------------------------------------------------------ forward
// Output tile 64x64 (e, r) with tile_e <= tile_r; wave w owns rows 16w..+15
// and four 16-column blocks; K = pixels [ks, ks + kchunk).
__device__ __forceinline__ void tri_tile(int t, int ntl, int &te, int &tr) {
    // enumerate (te, tr) with te <= tr row by row
    int a = 0;
    while (t >= ntl - a) {
        t -= ntl - a;
        ++a;
    }
    te = a;
    tr = a + t;
}

// Largest circular index distance min(|e - r|, m - |e - r|) over the pairs
// e in [e0, e0 + ne), r in [r0, r0 + nr): the distance is piecewise linear
// in r - e with its peaks at +-m/2, so the maximum is at an end of the
// difference range or at a peak inside it.
__device__ __forceinline__ int max_circ_dist(int m, int e0, int ne, int r0, int nr) {
    const int lo = r0 - (e0 + ne - 1), hi = (r0 + nr - 1) - e0;
    auto cd = [m](int d) {
        d = d < 0 ? -d : d;
        d %= m;
        return d < m - d ? d : m - d;
    };
    int best = cd(lo) > cd(hi) ? cd(lo) : cd(hi);
    const int h = m / 2;
    if ((lo <= h && h <= hi) || (lo <= -h && -h <= hi)) best = h;
    return best;
}

// A 32 x 32 (e, r) block of a tile whose value is never used: below the
// diagonal of a diagonal tile (the reduction reads e <= r), or, with
// dmin >= 32, every pair of the block closer than dmin (weighted by zero).
__device__ __forceinline__ bool fwd_block_idle(const FwdParams &P, int te, int tr, int we, int wr) {
    if (te == tr && we > wr) return true;
    return P.dmin >= 32 &&
           max_circ_dist(P.m, te * 64 + 32 * we, 32, tr * 64 + 32 * wr, 32) < P.dmin;
}

// FP64.  A 64 x 64 tile of pairs per workgroup, 16 pixels a step: the tile's
// rows go through LDS (two buffers, the next step's in registers meanwhile), as
// 128-byte runs of a row, so that L2 is asked for a row once per workgroup and
// not once per wave, and the MFMAs (64 cycles each) are what is left to wait
// for.  Of a tile on the diagonal one set of rows is staged and only the
// 16 x 16 blocks on or above it are formed; the waves take their 16 rows in
// another order in each split, so that the SIMDs share the shorter ones.  Two
// frequencies, with every wave loading its operands from memory and now: 64
// elements / 128^2 51 -> 30 us, 256 / 301x255 1695 -> 1002, 256 / 480^2 5.9 ->
// 2.87 ms (1.9 ms of MFMA time at 78.6 TFLOP/s).
constexpr int kFdT = 64, kFdPx = 16;        // tile, pixels a step
constexpr int kFdRow = kFdPx + 2;           // LDS row: 16 lanes' 16-byte reads hit 64 banks
typedef double fd2 __attribute__((ext_vector_type(2)));
typedef fd2 fd2_u __attribute__((aligned(8)));   // a row may start at any pixel

__global__ void __launch_bounds__(256) k_forward_f64(FwdParams P, const double *__restrict__ Gr,
                                                     const double *__restrict__ Gi,
                                                     const double *__restrict__ delta, double *__restrict__ part) {
    using acc_t = MM<double>::acc;
    __shared__ __align__(16) double buf[2][2][2][kFdT * kFdRow];   // step, side, re/im
    const int lane = threadIdx.x & 63;
    const int row = lane & 15, kk = lane >> 4;
    int te, tr;
    tri_tile(blockIdx.x, P.ntl, te, tr);
    const int split = blockIdx.y, k = blockIdx.z;
    const int wave = (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) + split) & 3;
    const int64_t N = P.N;
    const bool diag = te == tr;
    const int64_t ks = (int64_t)split * P.kchunk;
    const int64_t ke = std::min<int64_t>(N, ks + P.kchunk);
    const int c0 = diag ? wave : 0;   // first column block used

    // staging: thread t takes the pixel pair t % 8 of rows t / 8 and t / 8 + 32
    // of each side (rows at or beyond m: the last one, outputs never read)
    const int sp = 2 * (threadIdx.x & 7), sr = threadIdx.x >> 3;
    int64_t src[2][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        src[0][h] = ((int64_t)k * P.m + std::min(te * kFdT + sr + 32 * h, P.m - 1)) * N;
        src[1][h] = ((int64_t)k * P.m + std::min(tr * kFdT + sr + 32 * h, P.m - 1)) * N;
    }
    fd2 v[2][2][2];   // side, half, re/im
    auto load = [&](int64_t xc) {
        const int64_t x = xc + sp;
#pragma unroll
        for (int sd = 0; sd < 2; ++sd) {
            if (sd && diag) break;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const double *qr = Gr + src[sd][h], *qi = Gi + src[sd][h];
                if (xc + kFdPx <= N) {
                    v[sd][h][0] = *reinterpret_cast<const fd2_u *>(qr + x);
                    v[sd][h][1] = *reinterpret_cast<const fd2_u *>(qi + x);
                } else {   // the table's last pixels, then zeros
                    v[sd][h][0] = fd2{x < N ? qr[x] : 0.0, x + 1 < N ? qr[x + 1] : 0.0};
                    v[sd][h][1] = fd2{x < N ? qi[x] : 0.0, x + 1 < N ? qi[x + 1] : 0.0};
                }
            }
        }
    };
    auto store = [&](int b) {
#pragma unroll
        for (int sd = 0; sd < 2; ++sd) {
            if (sd && diag) break;
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int c = 0; c < 2; ++c)
                    *reinterpret_cast<fd2 *>(&buf[b][sd][c][(sr + 32 * h) * kFdRow + sp]) = v[sd][h][c];
        }
    };
    acc_t re[4], im[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) re[c] = im[c] = acc_t{0, 0, 0, 0};
    const int rs = diag ? 0 : 1;
    load(ks);
    store(0);
    int b = 0;
    for (int64_t xc = ks; xc < ke; xc += kFdPx, b ^= 1) {
        __syncthreads();   // buffer b is whole; every wave has left b ^ 1
        if (xc + kFdPx < ke) load(xc + kFdPx);
        double a_r[4], a_i[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int64_t x = xc + 4 * kk + s;
            const double dl = x < ke ? delta[x] : 0.0;
            const int o = (16 * wave + row) * kFdRow + 4 * kk + s;
            a_r[s] = buf[b][0][0][o] * dl;
            a_i[s] = buf[b][0][1][o] * dl;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (c < c0) continue;   // wave-uniform
            double b_r[4], b_i[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int o = (16 * c + row) * kFdRow + 4 * kk + s;
                b_r[s] = buf[b][rs][0][o];
                b_i[s] = buf[b][rs][1][o];
            }
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                re[c] = MM<double>::mma(a_r[s], b_r[s], re[c]);
                im[c] = MM<double>::mma(a_r[s], b_i[s], im[c]);
                re[c] = MM<double>::mma(-a_i[s], b_i[s], re[c]);
                im[c] = MM<double>::mma(a_i[s], b_r[s], im[c]);
            }
        }
        if (xc + kFdPx < ke) store(b ^ 1);
    }
    // partial tile -> part[split][k][e][r][2]
    double *pp = part + ((int64_t)split * P.nf + k) * P.mp * P.mp * 2;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        if (c < c0) continue;
        const int r = tr * kFdT + 16 * c + row;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int ee = te * kFdT + 16 * wave + MM<double>::out_row(kk, i);
            *reinterpret_cast<fd2_u *>(pp + ((int64_t)ee * P.mp + r) * 2) = fd2{re[c][i], im[c][i]};
        }
    }
}

// d[k][e][r] = c_k * sum_split part (fixed order) over the upper triangle
// e <= r, written to (e, r) and (r, e).  A block takes NT / RG entries of a
// row (grid: runs of them, rows, frequencies; runs below the diagonal exit); its
// RG thread groups each sum a contiguous part of the splits, eight loads in
// flight, and the group sums are added in order.  Eight groups where there are
// few entries: with one thread per entry the loop over the splits was a serial
// chain of load latencies (64 elements / 128^2: 122 us with 512 splits in FP64;
// the whole call 177 -> 51 us).  One group from kRedEntries entries on, which fill the
// card by themselves (1000 elements / 32^2, two frequencies, 13 splits: 151 -> 100 us a call, BF16 110 -> 52).
constexpr int64_t kRedEntries = 1 << 18;
struct FwdSplitOut {   // of k_forward_split, or null
    const uint8_t *flags;
    const float *scale, *dscale;
    int tile;
};
template <typename T, int RG, int NT>
__global__ void __launch_bounds__(NT) k_forward_reduce(FwdParams P, const T *__restrict__ part,
                                                               const float *__restrict__ gscale,
                                                               const double *__restrict__ dmax,
                                                               double *__restrict__ d, FwdSplitOut so) {
    constexpr int RN = NT / RG;   // entries
    __shared__ double s_r[RG][RN], s_i[RG][RN];
    const int t = threadIdx.x % RN, g = threadIdx.x / RN;
    const int k = blockIdx.z, e = blockIdx.y, r0 = blockIdx.x * RN, r = r0 + t;
    if (r0 + RN - 1 < e) return;   // block-uniform
    // (pairs closer than dmin are weighted by zero by the caller, and their
    // tile may not have been computed)
    const bool near = P.dmin >= 32 && min(abs(r - e), P.m - abs(r - e)) < P.dmin;
    const bool use = r >= e && r < P.m && !near;
    typedef T T2 __attribute__((ext_vector_type(2)));
    const int64_t stride = (int64_t)P.nf * P.mp * P.mp;   // one split
    const T2 *pp = reinterpret_cast<const T2 *>(part) + (int64_t)k * P.mp * P.mp + (int64_t)e * P.mp + r;
    double sr = 0.0, si = 0.0;
    // k_forward_split's partials carry the scales of their two rows, unless
    // the block of either is flagged
    double inv = 1.0, dsc = 1.0;
    const uint8_t *fe = nullptr, *fr = nullptr;
    if (so.flags && use) {
        inv = 1.0 / ((double)so.scale[k * P.m + e] * (double)so.scale[k * P.m + r]);
        dsc = 1.0 / (double)so.dscale[0];
        fe = so.flags + (int64_t)k * P.nsplit * P.ntl + e / so.tile;
        fr = so.flags + (int64_t)k * P.nsplit * P.ntl + r / so.tile;
    }
    constexpr int kU = 8;
    const int s1 = (int)((int64_t)P.nsplit * (g + 1) / RG);
    for (int s0 = (int)((int64_t)P.nsplit * g / RG); s0 < s1; s0 += kU) {
        T2 v[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) v[u] = use && s0 + u < s1 ? pp[(s0 + u) * stride] : T2{0, 0};
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const bool raw = fe && s0 + u < s1 && (fe[(s0 + u) * P.ntl] | fr[(s0 + u) * P.ntl]);
            const double f = raw ? 1.0 : inv;
            sr += (double)v[u][0] * f;
            si += (double)v[u][1] * f;
        }
    }
    s_r[g][t] = sr * dsc;
    s_i[g][t] = si * dsc;
    __syncthreads();
    if (g != 0 || r < e || r >= P.m) return;
    sr = si = 0.0;
#pragma unroll
    for (int q = 0; q < RG; ++q) {
        sr += s_r[q][t];
        si += s_i[q][t];
    }
    double c = P.cg[k];
    if (gscale) {
        const double gs = (double)gscale[k];
        c *= gs * gs;
    }
    if (dmax) c *= dmax[0];
    const double vr = sr * c, vi = si * c;
    const int64_t o1 = ((int64_t)k * P.m + e) * P.m + r, o2 = ((int64_t)k * P.m + r) * P.m + e;
    d[2 * o1] = vr;
    d[2 * o1 + 1] = vi;
    d[2 * o2] = vr;
    d[2 * o2 + 1] = vi;
}

// Workgroup -> (tile, split, frequency) for the flat grid of the 16-bit
// kernel.  The tiles of one pixel split read the same pixel range of G, so
// consecutive logical ids (tile fastest) are kept on one XCD and its L2.
__device__ __forceinline__ void fwd_block(const FwdParams &P, int &te, int &tr, int &split, int &k) {
    const int64_t nblk = (int64_t)P.ntri * P.nsplit * P.nf;
    const int64_t L = xcd_remap(blockIdx.x, nblk);
    const int t = (int)(L % P.ntri);
    const int64_t rest = L / P.ntri;
    split = (int)(rest % P.nsplit);
    k = (int)(rest / P.nsplit);
    tri_tile(t, P.ntl, te, tr);
}

// Forward, tables whose rows are not 16-byte aligned (N not a multiple of
// 4).  A 64 x 64 (e, r) output tile per workgroup (upper triangle only)
// over a split of the pixels; waves are 2 x 2, each 32 e x 32 r.  Pixels are
// consumed 32 at a time: G_e and G_r delta for the tile's rows are staged in
// LDS as [row][32 px] (stride 36), double buffered through registers; a
// lane reads its eight k values of a row as two b128 reads.
constexpr int kFwdKC = 32, kFwdLD = 36;

// One thread's staging registers: eight pixels of one row of G_e and of
// G_r, and delta at those pixels.  G_r delta is formed when the tile is
// stored, not when it is loaded, so the loads stay in flight during the
// MFMAs of the current tile.
struct FwdStage {
    f4 ar[2], ai[2], br[2], bi[2];
    double dl[8];
};

template <typename D>
__device__ __forceinline__ void fwd_stage_load(const float *__restrict__ gr, const float *__restrict__ gi,
                                               const D *__restrict__ delta, int m, int64_t N, int e_row,
                                               int r_row, int64_t xc, int64_t ke, bool vec, FwdStage &v) {
    const int c8 = (threadIdx.x & 3) * 8;
    const int64_t xs = xc + c8;
    if (vec) {
#pragma unroll
        for (int q = 0; q < 8; ++q) v.dl[q] = delta[xs + q];
        if (e_row < m) {
            const float *pr = gr + (int64_t)e_row * N + xs;
            const float *pi = gi + (int64_t)e_row * N + xs;
            v.ar[0] = *reinterpret_cast<const f4 *>(pr);
            v.ar[1] = *reinterpret_cast<const f4 *>(pr + 4);
            v.ai[0] = *reinterpret_cast<const f4 *>(pi);
            v.ai[1] = *reinterpret_cast<const f4 *>(pi + 4);
        } else {
            v.ar[0] = v.ar[1] = v.ai[0] = v.ai[1] = f4{0, 0, 0, 0};
        }
        if (r_row < m) {
            const float *pr = gr + (int64_t)r_row * N + xs;
            const float *pi = gi + (int64_t)r_row * N + xs;
            v.br[0] = *reinterpret_cast<const f4 *>(pr);
            v.br[1] = *reinterpret_cast<const f4 *>(pr + 4);
            v.bi[0] = *reinterpret_cast<const f4 *>(pi);
            v.bi[1] = *reinterpret_cast<const f4 *>(pi + 4);
        } else {
            v.br[0] = v.br[1] = v.bi[0] = v.bi[1] = f4{0, 0, 0, 0};
        }
    } else {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int64_t x = xs + q;
            const bool okx = x < ke;
            v.dl[q] = okx ? (double)delta[x] : 0.0;
            const bool oka = okx && e_row < m, okb = okx && r_row < m;
            v.ar[q >> 2][q & 3] = oka ? gr[(int64_t)e_row * N + x] : 0.0f;
            v.ai[q >> 2][q & 3] = oka ? gi[(int64_t)e_row * N + x] : 0.0f;
            v.br[q >> 2][q & 3] = okb ? gr[(int64_t)r_row * N + x] : 0.0f;
            v.bi[q >> 2][q & 3] = okb ? gi[(int64_t)r_row * N + x] : 0.0f;
        }
    }
}

template <typename D>
__device__ __forceinline__ void fwd_f32_regs_tile(const FwdParams &P, const float *__restrict__ Gr,
                                                  const float *__restrict__ Gi, const D *__restrict__ delta,
                                                  float *__restrict__ part, int te, int tr, int split, int k) {
    __shared__ float sA[2][2][64][kFwdLD];
    __shared__ float sBm[2][2][64][kFwdLD];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row = lane & 15, kk = lane >> 4;
    const int we = wave >> 1, wr = wave & 1;
    const int64_t N = P.N;
    const float *gr = Gr + (int64_t)k * P.m * N;
    const float *gi = Gi + (int64_t)k * P.m * N;
    const int64_t ks = (int64_t)split * P.kchunk;
    const int64_t ke = std::min<int64_t>(N, ks + P.kchunk);
    const int nch = (int)((ke - ks + kFwdKC - 1) / kFwdKC);
    const int srow = tid >> 2, c8 = (tid & 3) * 8;
    const int e_row = te * 64 + srow, r_row = tr * 64 + srow;
    // Waves whose block is never used only stage (wave-uniform); a tile
    // with no used block returns at once (the reduction does not read it).
    if (P.dmin >= 32 && max_circ_dist(P.m, te * 64, 64, tr * 64, 64) < P.dmin) return;
    const bool idle = fwd_block_idle(P, te, tr, we, wr);
    // (a + ib)(c + id) with three real products: P1 = ac, P2 = bd,
    // P3 = (a + b)(c + d); re = P1 - P2, im = P3 - P1 - P2
    f4 p1[2][2], p2[2][2], p3[2][2];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int c = 0; c < 2; ++c) p1[b][c] = p2[b][c] = p3[b][c] = f4{0, 0, 0, 0};
    auto vec_ok = [&](int64_t xc) { return ((N & 3) == 0) && (xc + kFwdKC <= ke); };
    auto store = [&](int buf, const FwdStage &stg) {
        *reinterpret_cast<f4 *>(&sA[buf][0][srow][c8]) = stg.ar[0];
        *reinterpret_cast<f4 *>(&sA[buf][0][srow][c8 + 4]) = stg.ar[1];
        *reinterpret_cast<f4 *>(&sA[buf][1][srow][c8]) = stg.ai[0];
        *reinterpret_cast<f4 *>(&sA[buf][1][srow][c8 + 4]) = stg.ai[1];
        f4 br0, br1, bi0, bi1;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            br0[q] = stg.br[0][q] * (float)stg.dl[q];
            br1[q] = stg.br[1][q] * (float)stg.dl[q + 4];
            bi0[q] = stg.bi[0][q] * (float)stg.dl[q];
            bi1[q] = stg.bi[1][q] * (float)stg.dl[q + 4];
        }
        *reinterpret_cast<f4 *>(&sBm[buf][0][srow][c8]) = br0;
        *reinterpret_cast<f4 *>(&sBm[buf][0][srow][c8 + 4]) = br1;
        *reinterpret_cast<f4 *>(&sBm[buf][1][srow][c8]) = bi0;
        *reinterpret_cast<f4 *>(&sBm[buf][1][srow][c8 + 4]) = bi1;
    };
    auto load = [&](int c, FwdStage &v) {
        const int64_t xc = ks + (int64_t)c * kFwdKC;
        fwd_stage_load(gr, gi, delta, P.m, N, e_row, r_row, xc, ke, vec_ok(xc), v);
    };
    // Tiles are loaded two steps ahead into two register sets used in turn
    // (as in the 16-bit kernel); FUT: tile c + 2 exists and is whole.
    auto step = [&](int c, FwdStage &next, FwdStage &fut, auto fut_tag) {
        const int buf = c & 1;
        if (decltype(fut_tag)::value)
            fwd_stage_load(gr, gi, delta, P.m, N, e_row, r_row, ks + (int64_t)(c + 2) * kFwdKC, ke, true, fut);
        else if (c + 2 < nch)
            load(c + 2, fut);
        if (!idle) {
        f4 a_r[2][2], a_i[2][2], b_r[2][2], b_i[2][2];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int ra = 32 * we + 16 * b + row;
            a_r[b][0] = *reinterpret_cast<const f4 *>(&sA[buf][0][ra][8 * kk]);
            a_r[b][1] = *reinterpret_cast<const f4 *>(&sA[buf][0][ra][8 * kk + 4]);
            a_i[b][0] = *reinterpret_cast<const f4 *>(&sA[buf][1][ra][8 * kk]);
            a_i[b][1] = *reinterpret_cast<const f4 *>(&sA[buf][1][ra][8 * kk + 4]);
            const int rb = 32 * wr + 16 * b + row;
            b_r[b][0] = *reinterpret_cast<const f4 *>(&sBm[buf][0][rb][8 * kk]);
            b_r[b][1] = *reinterpret_cast<const f4 *>(&sBm[buf][0][rb][8 * kk + 4]);
            b_i[b][0] = *reinterpret_cast<const f4 *>(&sBm[buf][1][rb][8 * kk]);
            b_i[b][1] = *reinterpret_cast<const f4 *>(&sBm[buf][1][rb][8 * kk + 4]);
        }
#pragma unroll
        for (int s8 = 0; s8 < 8; ++s8) {
            float ys[2];
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) ys[cb] = b_r[cb][s8 >> 2][s8 & 3] + b_i[cb][s8 >> 2][s8 & 3];
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const float xr = a_r[b][s8 >> 2][s8 & 3], xi = a_i[b][s8 >> 2][s8 & 3];
                const float xs = xr + xi;
#pragma unroll
                for (int cb = 0; cb < 2; ++cb) {
                    p1[b][cb] = MM<float>::mma(xr, b_r[cb][s8 >> 2][s8 & 3], p1[b][cb]);
                    p2[b][cb] = MM<float>::mma(xi, b_i[cb][s8 >> 2][s8 & 3], p2[b][cb]);
                    p3[b][cb] = MM<float>::mma(xs, ys[cb], p3[b][cb]);
                }
            }
        }
        }
        if (c + 1 < nch) store(buf ^ 1, next);
        __syncthreads();
    };
    FwdStage s0, s1;
    if (nch > 0) {
        load(0, s0);
        store(0, s0);
    }
    if (nch > 1) load(1, s1);
    __syncthreads();
    int c = 0;
    const int nwhole = ((N & 3) == 0) ? nch - 1 : 0;   // tiles 0 .. nch - 2 are whole
    for (; c + 4 <= nwhole; c += 2) {
        step(c, s1, s0, std::true_type());
        step(c + 1, s0, s1, std::true_type());
    }
    for (; c + 1 < nch; c += 2) {
        step(c, s1, s0, std::false_type());
        step(c + 1, s0, s1, std::false_type());
    }
    if (c < nch) step(c, s1, s0, std::false_type());
    float *pp = part + ((int64_t)split * P.nf + k) * P.mp * P.mp * 2;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
            const int r = tr * 64 + 32 * wr + 16 * cb + row;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int ee = te * 64 + 32 * we + 16 * b + MM<float>::out_row(kk, i);
                const int64_t o = ((int64_t)ee * P.mp + r) * 2;
                pp[o] = p1[b][cb][i] - p2[b][cb][i];
                pp[o + 1] = (p3[b][cb][i] - p1[b][cb][i]) - p2[b][cb][i];
            }
        }
    }
}

__global__ void __launch_bounds__(256, 2) k_forward_f32_regs(FwdParams P, const float *__restrict__ Gr,
                                                             const float *__restrict__ Gi,
                                                             const double *__restrict__ delta,
                                                             float *__restrict__ part) {
    int te, tr;
    tri_tile(blockIdx.x, P.ntl, te, tr);
    fwd_f32_regs_tile(P, Gr, Gi, delta, part, te, tr, blockIdx.y, blockIdx.z);
}

// Forward, FP32 tables with 16-byte aligned rows (N a multiple of 4).  The
// same tiles and waves as above, pixels consumed 16 at a time, and no
// staging registers: the tile rows of G_e and G_r (re, im) go from global
// memory straight into LDS (global_load_lds, 16 bytes per lane), double
// buffered, next to delta for the step's 16 pixels (as float, zero beyond
// N), and each wave scales its own B fragments by delta after reading them.
// Tile rows are 64 bytes, their four 16-byte chunks XOR-swizzled by
// (row / 2) mod 4 (a fragment read of 16 rows then meets no bank twice);
// a lane fills slot l mod 4 of row l / 4 and so loads the global chunk that
// the swizzle puts there.  Rows beyond m read row m - 1 and pixels beyond N
// read the row's last chunk: their outputs are never read, or delta is
// zero there.  With 32 KiB of LDS and about 100 registers a CU holds four
// workgroups; consecutive workgroups are the tiles of one pixel split
// on one XCD, which then reads each table row of the split from HBM about
// once.
constexpr int kFdKC = 16, kFdArr = 64 * 64, kFdBuf = 4 * kFdArr + 64;
constexpr int64_t kFdSplitPx = 16384;   // longest pixel split (1024 k-steps)
constexpr int64_t kWidePx = 900000;         // see fwd16_wide
constexpr int64_t kMinSplitPx = 64, kMinSplitPx32 = 16, kFewSplitPx = 512;   // shortest, see fwd_params
typedef __attribute__((address_space(3))) void lds_void_t;

__device__ __forceinline__ int fd_off(int row, int ch) { return row * 64 + 16 * (ch ^ ((row >> 1) & 3)); }

// out[x] = (float)delta[x] for x < N, 0 for N <= x < n
__global__ void k_delta_cast(int64_t N, int64_t n, const double *__restrict__ delta, float *__restrict__ out) {
    const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (x < n) out[x] = x < N ? (float)delta[x] : 0.0f;
}

// With O double the sums of each step (kFdKC pixels) are added in FP64, so that a
// split of any length is as exact as splits of a step whose partials are added in
// FP64, with fewer partials to write and read (see fwd_params).
template <typename O>
__device__ __forceinline__ void fwd_f32_tile(const FwdParams &P, const float *__restrict__ Gr,
                                             const float *__restrict__ Gi, const float *__restrict__ df,
                                             O *__restrict__ part, int te, int tr, int split, int k) {
    constexpr bool SUM64 = sizeof(O) == 8;
    __shared__ __align__(16) unsigned char sm[2][kFdBuf];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row = lane & 15, kk = lane >> 4;
    const int we = wave >> 1, wr = wave & 1;
    if (P.dmin >= 32 && max_circ_dist(P.m, te * 64, 64, tr * 64, 64) < P.dmin) return;
    const bool idle = fwd_block_idle(P, te, tr, we, wr);
    const int64_t N = P.N;
    const int64_t ks = (int64_t)split * P.kchunk;
    const int64_t ke = std::min<int64_t>(N, ks + P.kchunk);
    const int nch = (int)((ke - ks + kFdKC - 1) / kFdKC);
    // this lane's staging slot: tile row rl of each array, global chunk ch
    const int rl = 16 * wave + (lane >> 2);
    const int ch = (lane & 3) ^ ((rl >> 1) & 3);
    const int64_t go = (int64_t)k * P.m * N;
    const float *ae = Gr + go + (int64_t)std::min(te * 64 + rl, P.m - 1) * N;
    const float *ai = Gi + go + (int64_t)std::min(te * 64 + rl, P.m - 1) * N;
    const float *be = Gr + go + (int64_t)std::min(tr * 64 + rl, P.m - 1) * N;
    const float *bi = Gi + go + (int64_t)std::min(tr * 64 + rl, P.m - 1) * N;
    auto stage = [&](int c, int buf) {
        const int64_t xc = ks + (int64_t)c * kFdKC;
        const int64_t x = std::min<int64_t>(xc + 4 * ch, N - 4);
        unsigned char *d = sm[buf] + wave * 16 * 64;   // rows 16 wave .. 16 wave + 15
        __builtin_amdgcn_global_load_lds(ae + x, (lds_void_t *)d, 16, 0, 0);
        __builtin_amdgcn_global_load_lds(ai + x, (lds_void_t *)(d + kFdArr), 16, 0, 0);
        __builtin_amdgcn_global_load_lds(be + x, (lds_void_t *)(d + 2 * kFdArr), 16, 0, 0);
        __builtin_amdgcn_global_load_lds(bi + x, (lds_void_t *)(d + 3 * kFdArr), 16, 0, 0);
        if (lane == 0)   // delta at pixels xc + 4 wave .. + 3
            __builtin_amdgcn_global_load_lds(df + xc + 4 * wave, (lds_void_t *)(sm[buf] + 4 * kFdArr + 16 * wave),
                                             16, 0, 0);
    };
    // (a + ib)(c + id) with three real products: P1 = ac, P2 = bd,
    // P3 = (a + b)(c + d); re = P1 - P2, im = P3 - P1 - P2
    f4 p1[2][2], p2[2][2], p3[2][2];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int c = 0; c < 2; ++c) p1[b][c] = p2[b][c] = p3[b][c] = f4{0, 0, 0, 0};
    typedef double d4 __attribute__((ext_vector_type(4)));
    d4 tre[2][2], tim[2][2];   // with SUM64
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int c = 0; c < 2; ++c) tre[b][c] = tim[b][c] = d4{0, 0, 0, 0};
    auto add_step = [&]() {
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    tre[b][c][i] += (double)(p1[b][c][i] - p2[b][c][i]);
                    tim[b][c][i] += (double)((p3[b][c][i] - p1[b][c][i]) - p2[b][c][i]);
                }
                p1[b][c] = p2[b][c] = p3[b][c] = f4{0, 0, 0, 0};
            }
    };
    if (nch > 0) stage(0, 0);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    for (int c = 0; c < nch; ++c) {
        const int buf = c & 1;
        if (c + 1 < nch) stage(c + 1, buf ^ 1);
        if (!idle) {
            const unsigned char *sb = sm[buf];
            f4 a_r[2], a_i[2], b_r[2], b_i[2];
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const int ra = 32 * we + 16 * b + row, rb = 32 * wr + 16 * b + row;
                a_r[b] = *reinterpret_cast<const f4 *>(sb + fd_off(ra, kk));
                a_i[b] = *reinterpret_cast<const f4 *>(sb + kFdArr + fd_off(ra, kk));
                b_r[b] = *reinterpret_cast<const f4 *>(sb + 2 * kFdArr + fd_off(rb, kk));
                b_i[b] = *reinterpret_cast<const f4 *>(sb + 3 * kFdArr + fd_off(rb, kk));
            }
            const f4 dl = *reinterpret_cast<const f4 *>(sb + 4 * kFdArr + 16 * kk);
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
                b_r[cb] *= dl;
                b_i[cb] *= dl;
            }
#pragma unroll
            for (int s4 = 0; s4 < 4; ++s4) {
                float ys[2];
#pragma unroll
                for (int cb = 0; cb < 2; ++cb) ys[cb] = b_r[cb][s4] + b_i[cb][s4];
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    const float xr = a_r[b][s4], xi = a_i[b][s4];
                    const float xs = xr + xi;
#pragma unroll
                    for (int cb = 0; cb < 2; ++cb) {
                        p1[b][cb] = MM<float>::mma(xr, b_r[cb][s4], p1[b][cb]);
                        p2[b][cb] = MM<float>::mma(xi, b_i[cb][s4], p2[b][cb]);
                        p3[b][cb] = MM<float>::mma(xs, ys[cb], p3[b][cb]);
                    }
                }
            }
            if (SUM64) add_step();
        }
        __builtin_amdgcn_s_waitcnt(0);   // tile c + 1 has landed in LDS
        __syncthreads();
    }
    if (idle) return;
    O *pp = part + ((int64_t)split * P.nf + k) * P.mp * P.mp * 2;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
            const int r = tr * 64 + 32 * wr + 16 * cb + row;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int ee = te * 64 + 32 * we + 16 * b + MM<float>::out_row(kk, i);
                const int64_t o = ((int64_t)ee * P.mp + r) * 2;
                if (SUM64) {
                    pp[o] = tre[b][cb][i];
                    pp[o + 1] = tim[b][cb][i];
                } else {
                    pp[o] = p1[b][cb][i] - p2[b][cb][i];
                    pp[o + 1] = (p3[b][cb][i] - p1[b][cb][i]) - p2[b][cb][i];
                }
            }
        }
    }
}

template <typename O>
__global__ void __launch_bounds__(256, sizeof(O) == 8 ? 2 : 4) k_forward_f32(FwdParams P,
                                                                             const float *__restrict__ Gr,
                                                                             const float *__restrict__ Gi,
                                                                             const float *__restrict__ df,
                                                                             O *__restrict__ part) {
    int te, tr, split, k;
    fwd_block(P, te, tr, split, k);
    fwd_f32_tile(P, Gr, Gi, df, part, te, tr, split, k);
}

// byte offset of 16-byte chunk ch of row `row` in a tile of 64-byte rows
__device__ __forceinline__ int f16_off(int row, int ch) { return row * 64 + 16 * (ch ^ ((row >> 1) & 3)); }

// ------------------------------------------------------------------ FP32 tables on the FP16 matrix cores
// Forward with FP32 tables, both operands split into two FP16 pieces (x s =
// hi + 2^-11 lo, s a power of two) and hi hi + 2^-11 (hi lo + lo hi) accumulated
// in FP32 on the 16x16x32 FP16 cores.
//
// FP16 holds x s to FP32's accuracy only between kFsMin (below, the low piece
// runs out of bits) and kFsMax.  What has to lie there is what the sums
// contain: delta (brought below 1 by its largest magnitude) is dealt to both
// sides, u = 2^round(log2 |delta| / 2) to G_e and delta / u to G_r, so that where
// delta is zero G does not count at all, and where it is small each operand
// shrinks only by its square root.  Row r of G at frequency k is scaled by its
// largest |G| sqrt(|delta|) over kFsSamples sampled pixels (2^8 there, 2^8 of
// headroom above and 2^21 below).  One workgroup per block of 128 rows, split and
// frequency looks whether every value of the block but zero lies in the range
// (testing all that is staged cost 73 of 849 us at 256 elements / 480^2); if not,
// the block is put on a list and flagged, and k_forward_f32_list computes its
// tiles from FP32 (unscaled partials, which the reduction tells by the flag).  A
// split with a delta below kFsDelta, which brings most values of G below the
// range, goes to the list at once.
//
// A 128 x 128 (e, r) tile per workgroup of eight waves, 4 x 2 of 32 x 64, 32
// pixels per k-step.  A step's 256 rows of G (128 bytes each and array) pass
// through registers, are scaled (those of the r side times delta) and split
// there, and stored as eight FP16 arrays of 8 KB, double buffered (128 KB: one
// workgroup per compute unit, two waves per SIMD).  During a step a wave
// multiplies, and converts its part of the next step's rows, which it loaded a
// step earlier, and loads that of the one after: waves 0 to 3 convert first
// and waves 4 to 7, which share their SIMDs, multiply first, so that the matrix
// cores work while vector instructions convert.
//
// 1024 elements / 1100^2, four frequencies: 130.2 ms on the FP32 cores, 68.5
// here (12 MFMAs per complex product of blocks: 0.91 PFLOP/s, the matrix cores busy
// 0.44 of the time at 2.0 GHz); 256 / 480^2, three frequencies: 1.36 -> 0.78 ms; 1024 /
// 255x301 (rows not 16-byte aligned), two: 11.6 -> 2.2 ms.  Relative L2 error
// against FP64, ordered pairs on the FP32 cores and so: 256 / 480^2 4.7e-7 -> 1.0e-7, 97 /
// 301x255 1.2e-7 -> 4.8e-8.  Four waves of 64 x 64 with 512 registers each spilled:
// the compiler moved accumulators between register files at every step.
constexpr int kFsT = 128, kFsKC = 32, kFsArr = kFsT * kFsKC * 2, kFsSamples = 256;
constexpr int kFsTop = 8;
constexpr float kFsMax = 65504.0f;      // largest FP16 value
constexpr float kFsMin = 0x1p-13f;      // steps of 2^-24 2^-11 are 2^-22 of it
constexpr float kFsDelta = 0x1p-42f;    // u = 2^-21
constexpr float kFsLo = 0x1p11f;        // scale of the low pieces
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef float f2 __attribute__((ext_vector_type(2)));

// The power of two that brings `top` > 0 into [2^(e-1), 2^e) (1 otherwise).
__device__ __forceinline__ float fs_scale(float top, int e) {
    if (!(top > 0.0f)) return 1.0f;
    int x;
    (void)frexpf(fminf(top, 3.0e38f), &x);
    return ldexpf(1.0f, min(max(e - x, -100), 100));
}

// Blocks 0 .. rows - 1: scale[row] of the rows (k m + r) = the largest |G|
// sqrt(|delta|) over the sampled pixels, or, if that is zero, minus the largest
// |G|.  The other blocks: partial maxima of |delta| (kReduceBlocks of them).
__global__ void __launch_bounds__(256) k_fs_scales(int64_t N, int rows, const float *__restrict__ Gr,
                                                   const float *__restrict__ Gi, const double *__restrict__ delta,
                                                   float *__restrict__ scale, float *__restrict__ dpart) {
    __shared__ float sm[4], sg[4];
    float v = 0.0f, g = 0.0f;
    if ((int)blockIdx.x < rows) {
        const int64_t x = (int64_t)threadIdx.x * N / kFsSamples, o = (int64_t)blockIdx.x * N + x;
        g = fmaxf(fabsf(Gr[o]), fabsf(Gi[o]));
        v = g * sqrtf(fabsf((float)delta[x]));
    } else {
        for (int64_t i = (int64_t)(blockIdx.x - rows) * 256 + threadIdx.x; i < N; i += kReduceBlocks * 256)
            v = fmaxf(v, fabsf((float)delta[i]));
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        v = fmaxf(v, __shfl_xor(v, o));
        g = fmaxf(g, __shfl_xor(g, o));
    }
    if ((threadIdx.x & 63) == 0) {
        sm[threadIdx.x >> 6] = v;
        sg[threadIdx.x >> 6] = g;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        v = fmaxf(fmaxf(sm[0], sm[1]), fmaxf(sm[2], sm[3]));
        g = fmaxf(fmaxf(sg[0], sg[1]), fmaxf(sg[2], sg[3]));
        if ((int)blockIdx.x < rows)
            scale[blockIdx.x] = v > 0.0f ? v : -g;
        else
            dpart[blockIdx.x - rows] = v;
    }
}

// df[x] = (float)delta[x] sd (zero from N to n), sd = fs_scale(max |delta|, 0)
// to dscale[0]; the rows' scales from their samples (2^100 for a row that is
// zero at every sampled pixel); clears the list and the flags.
__global__ void __launch_bounds__(256) k_fs_delta(int64_t N, int64_t n, const double *__restrict__ delta,
                                                  const float *__restrict__ dpart, float *__restrict__ df,
                                                  float *__restrict__ dscale, int rows, float *__restrict__ scale,
                                                  int *__restrict__ redo, uint8_t *__restrict__ flags,
                                                  int64_t nflags) {
    __shared__ float sm[4];
    float v = 0.0f;
#pragma unroll
    for (int q = 0; q < kReduceBlocks / 256; ++q) v = fmaxf(v, dpart[q * 256 + threadIdx.x]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = v;
    __syncthreads();
    const float sd = fs_scale(fmaxf(fmaxf(sm[0], sm[1]), fmaxf(sm[2], sm[3])), 0);
    const int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (x == 0) {
        dscale[0] = sd;
        redo[0] = 0;
    }
    if (x < n) df[x] = x < N ? (float)delta[x] * sd : 0.0f;
    for (int64_t q = x; q < rows; q += (int64_t)gridDim.x * 256) {
        const float t = scale[q];
        scale[q] = t > 0.0f ? fs_scale(t * sqrtf(sd), kFsTop) : (t < 0.0f ? fs_scale(-t, kFsTop) : 0x1p100f);
    }
    for (int64_t q = x; q < nflags; q += (int64_t)gridDim.x * 256) flags[q] = 0;
}

__global__ void __launch_bounds__(512, 2) k_forward_split(FwdParams P, const float *__restrict__ Gr,
                                                          const float *__restrict__ Gi,
                                                          const float *__restrict__ df,
                                                          const float *__restrict__ scale, float *__restrict__ part,
                                                          int *__restrict__ redo, uint8_t *__restrict__ flags) {
    using M = MM16<__half>;
    // [buffer][e re hi, e im hi, e re lo, e im lo, then the r side]
    __shared__ __align__(16) unsigned char sT[2][8 * kFsArr];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row = lane & 15, kk = lane >> 4;
    int te, tr, split, k;
    fwd_block(P, te, tr, split, k);
    // Rows 32 we, columns 64 wr of the tile.  Waves s and s + 4 share a SIMD: on
    // the diagonal, where two of the eight blocks lie below it and two need
    // half of their columns (the upper ones), these are dealt so that no SIMD has
    // more than one and a half (two, before): 128 elements / 480^2, two
    // frequencies, 204 -> 191 us, 97 / 301x255 80 -> 75; from 200 elements on, where
    // power limits the matrix cores, no difference.
    const int dw = (0x71326054 >> (4 * wave)) & 15;   // we + 4 wr
    const int we = te == tr ? dw & 3 : wave & 3, wr = te == tr ? dw >> 2 : wave >> 2;
    const bool upper = te == tr && (we == 1 + 2 * wr);
    if (P.dmin >= 32 && max_circ_dist(P.m, te * kFsT, kFsT, tr * kFsT, kFsT) < P.dmin) return;
    const bool idle = (te == tr && 32 * we >= 64 * (wr + 1)) ||
                      (P.dmin >= 32 && max_circ_dist(P.m, te * kFsT + 32 * we, 32, tr * kFsT + 64 * wr, 64) < P.dmin);
    const int64_t N = P.N;
    const int64_t ks = (int64_t)split * P.kchunk;
    const int64_t ke = std::min<int64_t>(N, ks + P.kchunk);
    const int last = (int)((ke - ks + kFsKC - 1) / kFsKC) - 1;   // last chunk
    // staging: pixels p4 .. p4 + 3 of rows r8, r8 + 64 of either side.  Rows
    // at or beyond m read row m - 1 (their outputs are never read), pixels at
    // or beyond N the last ones of the row (delta is zero there; the other
    // splits end with a whole chunk).
    const int p4 = (tid & 7) * 4, r8 = tid >> 3;
    const float *rowp[4];     // e rows, then r rows
    float sc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int r = std::min((j < 2 ? te : tr) * kFsT + r8 + 64 * (j & 1), P.m - 1);
        rowp[j] = Gr + ((int64_t)k * P.m + r) * N;
        sc[j] = scale[k * P.m + r];
    }
    const int64_t im = Gi - Gr;
    f4 v[4][2], dl;
    // Which workgroup looks at block b: its tile with the first of the blocks b,
    // b + 1, .. (around the ring) that is not skipped above.
    auto owner = [&](int b, int other) {
        for (int d = 0; d < P.ntl; ++d) {
            const int x = b + d < P.ntl ? b + d : b + d - P.ntl;
            if (x == other) return true;
            if (P.dmin < 32 || max_circ_dist(P.m, std::min(b, x) * kFsT, kFsT, std::max(b, x) * kFsT, kFsT) >= P.dmin)
                return false;
        }
        return false;
    };
    const bool own_e = owner(te, tr), own_r = te != tr && owner(tr, te);
    // of the values looked at (largest of re and im): the largest, and the bits
    // of the smallest but zero, minus one.  The other side's are less than twice
    // as large or half as small.
    float top[2] = {0.0f, 0.0f};
    unsigned low[2] = {0xffffffffu, 0xffffffffu};
    typedef f4 f4_a4 __attribute__((aligned(4)));   // rows need no alignment
    auto load = [&](int c) {
        const int64_t xc = ks + (int64_t)c * kFsKC + p4;
        if (xc - p4 + kFsKC <= N) {   // workgroup-uniform
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v[j][0] = *reinterpret_cast<const f4_a4 *>(rowp[j] + xc);
                v[j][1] = *reinterpret_cast<const f4_a4 *>(rowp[j] + im + xc);
            }
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int64_t x = std::min<int64_t>(xc + q, N - 1);
                    v[j][0][q] = rowp[j][x];
                    v[j][1][q] = rowp[j][im + x];
                }
        }
        dl = *reinterpret_cast<const f4 *>(df + xc);
    };
    auto store = [&](unsigned char *buf) {
        f4 du, dq;   // u and delta / u
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const unsigned ub = (((__float_as_uint(dl[q]) & 0x7f800000u) + 0x40000000u) >> 1) & 0x7f800000u;
            du[q] = dl[q] != 0.0f ? __uint_as_float(ub) : 0.0f;
            dq[q] = dl[q] * __uint_as_float(0x7f000000u - ub);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const f4 s = (j < 2 ? du : dq) * sc[j];
            f4 w[2];
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                w[a] = v[j][a] * s;
                const h4 h = __builtin_convertvector(w[a], h4);
                f4 rem;
#pragma unroll
                for (int q = 0; q < 4; ++q) rem[q] = (w[a][q] - (float)h[q]) * kFsLo;
                const h4 l = __builtin_convertvector(rem, h4);
                unsigned char *d =
                    buf + ((j < 2 ? 0 : 4) + a) * kFsArr + f16_off(r8 + 64 * (j & 1), p4 >> 3) + 2 * (p4 & 4);
                *reinterpret_cast<h4 *>(d) = h;
                *reinterpret_cast<h4 *>(d + 2 * kFsArr) = l;
            }
            if (j < 2 ? own_e : own_r) {   // workgroup-uniform
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float m = fmaxf(fabsf(w[0][q]), fabsf(w[1][q]));
                    top[j >> 1] = fmaxf(top[j >> 1], m);
                    low[j >> 1] = min(low[j >> 1], __float_as_uint(m) - 1u);
                }
            }
        }
    };
    f4 re[2][4], imv[2][4];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int c = 0; c < 4; ++c) re[b][c] = imv[b][c] = f4{0, 0, 0, 0};
    auto frag = [&](const unsigned char *q, int r) { return *reinterpret_cast<const h8 *>(q + f16_off(r, kk)); };
    auto mma = [&](const unsigned char *sa, const unsigned char *sb, auto c0) {
        h8 a[4][2], n[2][2];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
#pragma unroll
            for (int t = 0; t < 4; ++t) a[t][b] = frag(sa + t * kFsArr, 32 * we + 16 * b + row);
            n[0][b] = neg(a[1][b]);
            n[1][b] = neg(a[3][b]);
        }
#pragma unroll
        for (int cb = decltype(c0)::value; cb < 4; ++cb) {
            h8 u[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) u[t] = frag(sb + t * kFsArr, 64 * wr + 16 * cb + row);
            // (ar + i ai)(br + i bi) = ar br - ai bi + i (ar bi + ai br)
            // A step's products are summed by themselves, the hi lo ones first,
            // and added once: in the long sums over pixels it is the number of
            // roundings at the sum's own size that sets the error.
            f4 tr_[2], ti_[2];
#pragma unroll
            for (int b = 0; b < 2; ++b) tr_[b] = ti_[b] = f4{0, 0, 0, 0};
            auto term = [&](const h8 (&x)[2], const h8 &p, const h8 (&y)[2], const h8 &q) {
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    tr_[b] = M::mma(x[b], p, tr_[b]);
                    ti_[b] = M::mma(y[b], q, ti_[b]);
                }
            };
            term(a[0], u[2], a[0], u[3]);
            term(n[0], u[3], a[1], u[2]);
            term(a[2], u[0], a[2], u[1]);
            term(n[1], u[1], a[3], u[0]);
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                tr_[b] *= 1.0f / kFsLo;
                ti_[b] *= 1.0f / kFsLo;
            }
            term(a[0], u[0], a[0], u[1]);
            term(n[0], u[1], a[1], u[0]);
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                re[b][cb] += tr_[b];
                imv[b][cb] += ti_[b];
            }
        }
    };
    // the deltas of the split
    bool tiny = false;
    for (int64_t x = ks + tid; x < ke; x += 512) {
        const float d = fabsf(df[x]);
        tiny |= d > 0.0f && d < kFsDelta;
    }
    auto list = [&](int b) {
        const int id = (k * P.nsplit + split) * P.ntl + b;
        flags[id] = 1;
        redo[1 + atomicAdd(redo, 1)] = id;
    };
    if (__syncthreads_or(tiny)) {
        if (tid == 0) {
            if (own_e) list(te);
            if (own_r) list(tr);
        }
        return;
    }
    load(0);
    store(sT[0]);
    load(std::min(1, last));
    auto kloop = [&](auto first, auto c0) {   // first: convert before multiplying
        for (int c = 0; c <= last; ++c) {
            lds_barrier();   // chunk c is in LDS, and no wave still reads the other buffer
            const unsigned char *sa = sT[c & 1];
            unsigned char *sn = sT[(c & 1) ^ 1];
            // (the last two steps convert and load the last chunk again, unused)
            if (decltype(first)::value) {
                store(sn);
                load(std::min(c + 2, last));
                __builtin_amdgcn_sched_barrier(0);
            }
            if (!idle) mma(sa, sa + 4 * kFsArr, c0);
            if (!decltype(first)::value) {
                __builtin_amdgcn_sched_barrier(0);
                store(sn);
                load(std::min(c + 2, last));
            }
        }
    };
    typedef std::integral_constant<int, 0> C0;
    typedef std::integral_constant<int, 2> C2;
    if (wave < 4)
        kloop(std::true_type(), C0());
    else if (!upper)
        kloop(std::false_type(), C0());
    else
        kloop(std::false_type(), C2());
#pragma unroll
    for (int sd = 0; sd < 2; ++sd) {
        if (!(sd ? own_r : own_e)) continue;
        const int beyond =
            __syncthreads_or(!(top[sd] < 0.5f * kFsMax) || low[sd] < __float_as_uint(2.0f * kFsMin) - 1u);
        if (beyond && tid == 0) list(sd ? tr : te);
    }
    if (idle) return;
    float *pp = part + ((int64_t)split * P.nf + k) * P.mp * P.mp * 2;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
            const int r = tr * kFsT + 64 * wr + 16 * cb + row;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int ee = te * kFsT + 32 * we + 16 * b + 4 * kk + i;
                *reinterpret_cast<f2 *>(pp + ((int64_t)ee * P.mp + r) * 2) = f2{re[b][cb][i], imv[b][cb][i]};
            }
        }
    }
}

// The listed (block of rows, split, frequency)s of k_forward_split from FP32: each
// is ntl tiles, each of three or four 64 x 64 tiles.  Partials in units of
// (float)delta sd, G unscaled.  VEC: rows of whole 16-byte pieces (N a multiple
// of 4).
template <bool VEC>
__global__ void __launch_bounds__(256, 2) k_forward_f32_list(FwdParams P, const float *__restrict__ Gr,
                                                             const float *__restrict__ Gi,
                                                             const float *__restrict__ df,
                                                             float *__restrict__ part, const int *__restrict__ redo,
                                                             const uint8_t *__restrict__ flags) {
    const int64_t per = 4 * P.ntl, n = per * redo[0];
    for (int64_t i = blockIdx.x; i < n; i += gridDim.x) {
        const int id = redo[1 + i / per], q = (int)(i % per);
        const int rest = id / P.ntl, b = id - rest * P.ntl, x = q >> 2;
        // (a tile of two listed blocks is the lower one's)
        if (x < b && flags[rest * P.ntl + x]) continue;   // workgroup-uniform
        const int split = rest % P.nsplit, k = rest / P.nsplit;
        const int e64 = 2 * std::min(b, x) + ((q >> 1) & 1), r64 = 2 * std::max(b, x) + (q & 1);
        if (e64 <= r64) {
            if (VEC)
                fwd_f32_tile(P, Gr, Gi, df, part, e64, r64, split, k);
            else
                fwd_f32_regs_tile(P, Gr, Gi, df, part, e64, r64, split, k);
        }
        __syncthreads();   // the next item reuses the LDS
    }
}

// ------------------------------------------------------------------ 16-bit, LDS-staged
// Forward with 16-bit tables on the 16x16x32 matrix cores (FP32
// accumulation), tiled as the FP32 kernel: a 64 x 64 (e, r) tile per
// workgroup, waves 2 x 2 of 32 x 32, 32 pixels per k-step.  Both operands
// take eight consecutive pixels of one row per lane, which the tables store
// contiguously, so a thread stages eight pixels of one row of G_e and of
// G_r delta (delta pre-scaled to float) with 16-byte loads, and a fragment
// is one 16-byte LDS read.  The four 16-byte chunks of a 64-byte tile row
// are XOR-swizzled by (row / 2) mod 4, which puts the reads of a fragment
// on distinct banks.  Tiles are double buffered.
constexpr int kF16KC = 32, kF16Arr = 64 * kF16KC * 2;   // one array of a tile (bytes)

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// out[x] = delta[x] / max |delta| as float (0 if delta is zero), 0 for N <= x < n
__global__ void k_delta_f32(int64_t N, int64_t n, const double *__restrict__ delta, const double *__restrict__ dmax,
                            float *__restrict__ out) {
    const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= n) return;
    const double inv = dmax[0] > 0.0 ? 1.0 / dmax[0] : 0.0;
    out[x] = x < N ? (float)(delta[x] * inv) : 0.0f;
}

struct F16Stage {
    u32x4 ar, ai, br, bi;
    f4 d0, d1;
};

__device__ __forceinline__ void f16_stage_load(const unsigned short *__restrict__ gr,
                                               const unsigned short *__restrict__ gi,
                                               const float *__restrict__ df, int m, int64_t N, int e_row,
                                               int r_row, int64_t xs, int64_t ke, bool vec, F16Stage &v) {
    const u32x4 z = {0u, 0u, 0u, 0u};
    if (vec) {
        v.ar = e_row < m ? *reinterpret_cast<const u32x4 *>(gr + (int64_t)e_row * N + xs) : z;
        v.ai = e_row < m ? *reinterpret_cast<const u32x4 *>(gi + (int64_t)e_row * N + xs) : z;
        v.br = r_row < m ? *reinterpret_cast<const u32x4 *>(gr + (int64_t)r_row * N + xs) : z;
        v.bi = r_row < m ? *reinterpret_cast<const u32x4 *>(gi + (int64_t)r_row * N + xs) : z;
        v.d0 = *reinterpret_cast<const f4 *>(df + xs);
        v.d1 = *reinterpret_cast<const f4 *>(df + xs + 4);
    } else {
        unsigned short a_r[8], a_i[8], b_r[8], b_i[8];
        float d[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int64_t x = xs + q;
            const bool okx = x < ke;
            const bool oka = okx && e_row < m, okb = okx && r_row < m;
            a_r[q] = oka ? gr[(int64_t)e_row * N + x] : (unsigned short)0;
            a_i[q] = oka ? gi[(int64_t)e_row * N + x] : (unsigned short)0;
            b_r[q] = okb ? gr[(int64_t)r_row * N + x] : (unsigned short)0;
            b_i[q] = okb ? gi[(int64_t)r_row * N + x] : (unsigned short)0;
            d[q] = okx ? df[x] : 0.0f;
        }
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            v.ar[h] = a_r[2 * h] | ((unsigned)a_r[2 * h + 1] << 16);
            v.ai[h] = a_i[2 * h] | ((unsigned)a_i[2 * h + 1] << 16);
            v.br[h] = b_r[2 * h] | ((unsigned)b_r[2 * h + 1] << 16);
            v.bi[h] = b_i[2 * h] | ((unsigned)b_i[2 * h + 1] << 16);
        }
        v.d0 = f4{d[0], d[1], d[2], d[3]};
        v.d1 = f4{d[4], d[5], d[6], d[7]};
    }
}

// eight 16-bit values times delta, rounded back to the storage type
template <typename S, typename V>
__device__ __forceinline__ u32x4 f16_scale(u32x4 raw, f4 d0, f4 d1) {
    const V v = __builtin_bit_cast(V, raw);
    V o;
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = MM16<S>::from_f((float)v[i] * (i < 4 ? d0[i] : d1[i - 4]));
    return __builtin_bit_cast(u32x4, o);
}

template <typename S>
__global__ void __launch_bounds__(256, 2) k_forward16_lds(FwdParams P, const S *__restrict__ Gr,
                                                          const S *__restrict__ Gi, const float *__restrict__ df,
                                                          float *__restrict__ part) {
    using V = typename MM16<S>::vec;
    __shared__ __align__(16) unsigned char sA[2][2 * kF16Arr];   // [buffer][re, im] G_e rows
    __shared__ __align__(16) unsigned char sB[2][2 * kF16Arr];   // [buffer][re, im] G_r delta rows
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row = lane & 15, kk = lane >> 4;
    const int we = wave >> 1, wr = wave & 1;
    int te, tr, split, k;
    fwd_block(P, te, tr, split, k);
    const int64_t N = P.N;
    const unsigned short *gr = reinterpret_cast<const unsigned short *>(Gr + (int64_t)k * P.m * N);
    const unsigned short *gi = reinterpret_cast<const unsigned short *>(Gi + (int64_t)k * P.m * N);
    const int64_t ks = (int64_t)split * P.kchunk;
    const int64_t ke = std::min<int64_t>(N, ks + P.kchunk);
    const int nch = (int)((ke - ks + kF16KC - 1) / kF16KC);
    const int srow = tid >> 2, sch = tid & 3;
    const int e_row = te * 64 + srow, r_row = tr * 64 + srow;
    const int so = f16_off(srow, sch);
    // waves whose block is never used only stage (see k_forward_f32)
    if (P.dmin >= 32 && max_circ_dist(P.m, te * 64, 64, tr * 64, 64) < P.dmin) return;
    const bool idle = fwd_block_idle(P, te, tr, we, wr);
    f4 re[2][2], im[2][2];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int c = 0; c < 2; ++c) re[b][c] = im[b][c] = f4{0, 0, 0, 0};
    auto vec_ok = [&](int64_t xc) { return ((N & 7) == 0) && (xc + kF16KC <= ke); };
    auto load = [&](int c, F16Stage &v) {
        const int64_t xc = ks + (int64_t)c * kF16KC;
        f16_stage_load(gr, gi, df, P.m, N, e_row, r_row, xc + 8 * sch, ke, vec_ok(xc), v);
    };
    auto store = [&](int buf, const F16Stage &v) {
        *reinterpret_cast<u32x4 *>(sA[buf] + so) = v.ar;
        *reinterpret_cast<u32x4 *>(sA[buf] + kF16Arr + so) = v.ai;
        *reinterpret_cast<u32x4 *>(sB[buf] + so) = f16_scale<S, V>(v.br, v.d0, v.d1);
        *reinterpret_cast<u32x4 *>(sB[buf] + kF16Arr + so) = f16_scale<S, V>(v.bi, v.d0, v.d1);
    };
    // Tiles are loaded two steps ahead into two register sets used in turn:
    // step c computes on tile c (LDS), issues the loads of tile c + 2 and
    // stores tile c + 1, loaded a step earlier, to the other buffer.  Each
    // load then has two steps of MFMAs to arrive in.
    // FUT: tile c + 2 exists and is whole (16-byte loads, no tests), so the
    // steady state has unconditional loads and exact load-counter waits.
    auto step = [&](int c, F16Stage &next, F16Stage &fut, auto fut_tag) {
        const int buf = c & 1;
        if (decltype(fut_tag)::value)
            f16_stage_load(gr, gi, df, P.m, N, e_row, r_row, ks + (int64_t)(c + 2) * kF16KC + 8 * sch, ke, true,
                           fut);
        else if (c + 2 < nch)
            load(c + 2, fut);
        if (!idle) {
            V a_r[2], a_i[2], a_n[2], b_r[2], b_i[2];
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const int ra = 32 * we + 16 * b + row, rb = 32 * wr + 16 * b + row;
                a_r[b] = *reinterpret_cast<const V *>(sA[buf] + f16_off(ra, kk));
                a_i[b] = *reinterpret_cast<const V *>(sA[buf] + kF16Arr + f16_off(ra, kk));
                a_n[b] = neg(a_i[b]);
                b_r[b] = *reinterpret_cast<const V *>(sB[buf] + f16_off(rb, kk));
                b_i[b] = *reinterpret_cast<const V *>(sB[buf] + kF16Arr + f16_off(rb, kk));
            }
            // (ar + i ai)(br + i bi) = ar br - ai bi + i (ar bi + ai br)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int cb = 0; cb < 2; ++cb) {
                    re[b][cb] = MM16<S>::mma(a_r[b], b_r[cb], re[b][cb]);
                    re[b][cb] = MM16<S>::mma(a_n[b], b_i[cb], re[b][cb]);
                    im[b][cb] = MM16<S>::mma(a_r[b], b_i[cb], im[b][cb]);
                    im[b][cb] = MM16<S>::mma(a_i[b], b_r[cb], im[b][cb]);
                }
        }
        if (c + 1 < nch) store(buf ^ 1, next);
        __syncthreads();
    };
    F16Stage s0, s1;
    if (nch > 0) {
        load(0, s0);
        store(0, s0);
    }
    if (nch > 1) load(1, s1);
    __syncthreads();
    int c = 0;
    // tiles 0 .. nch - 2 are whole; the last may be partial
    const int nwhole = ((N & 7) == 0) ? nch - 1 : 0;
    for (; c + 4 <= nwhole; c += 2) {
        step(c, s1, s0, std::true_type());       // tile c + 1 in s1, tile c + 2 into s0
        step(c + 1, s0, s1, std::true_type());   // tile c + 2 in s0, tile c + 3 into s1
    }
    for (; c + 1 < nch; c += 2) {
        step(c, s1, s0, std::false_type());
        step(c + 1, s0, s1, std::false_type());
    }
    if (c < nch) step(c, s1, s0, std::false_type());
    float *pp = part + ((int64_t)split * P.nf + k) * P.mp * P.mp * 2;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
            const int r = tr * 64 + 32 * wr + 16 * cb + row;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int ee = te * 64 + 32 * we + 16 * b + 4 * kk + i;
                const int64_t o = ((int64_t)ee * P.mp + r) * 2;
                pp[o] = re[b][cb][i];
                pp[o + 1] = im[b][cb][i];
            }
        }
    }
}

// ------------------------------------------------------------------ 16-bit, wide tiles
// Forward with 16-bit tables, tiles of 256 (e) x 128 (r) by eight waves of 64 x
// 64 (4 x 4 blocks of 16 x 16, 64 MFMAs per wave and step of 32 pixels): 48 KB
// of operands per 512 MFMAs, where the 64 x 64 tiles above move 16 KB per 64.
// One workgroup per compute unit, two waves per SIMD.  A step's rows (64 bytes
// each and array) pass through registers, those of the r side times delta and
// rounded back to the storage type, into double-buffered LDS; as in
// k_forward_split a wave loads its part two steps ahead, and the two waves of
// a SIMD convert and multiply at different times.  Rows need no alignment.
// 1024 elements / 1100^2, four frequencies: 34.9 ms, as the 128 x 128 tiles it
// replaces (27.3 ms and 8.1 for their table of G delta, which it does not need:
// 19 GB of workspace less).  L2 requests bound it: rows lie megabytes apart, so
// a step takes 64-byte pieces, 81 G/s of them, with the matrix cores busy 0.26
// at 2.4 GHz; 128 x 128 tiles in steps of 64 pixels, loaded two steps ahead,
// took 65 ms.
constexpr int kWE = 256, kWR = 128;
constexpr int kWArrE = kWE * 64, kWArrR = kWR * 64;   // one array of a side (bytes)
constexpr int kWBuf = 2 * kWArrE + 2 * kWArrR;        // e re, e im, r re, r im
typedef u32x4 u32x4_a2 __attribute__((aligned(2)));

// tile (te, tr), split and frequency of a workgroup: consecutive logical ids are
// the tiles of one pixel split (see fwd_block)
__device__ __forceinline__ void wide_block(const FwdParams &P, int &te, int &tr, int &split, int &k) {
    const int64_t L = xcd_remap(blockIdx.x, gridDim.x);
    int t = (int)(L % P.ntri);
    const int64_t rest = L / P.ntri;
    split = (int)(rest % P.nsplit);
    k = (int)(rest / P.nsplit);
    te = 0;
    while (t >= P.ntl - 2 * te) t -= P.ntl - 2 * te++;
    tr = 2 * te + t;
}

template <typename S>
__global__ void __launch_bounds__(512, 2) k_forward16_wide(FwdParams P, const S *__restrict__ Gr,
                                                           const S *__restrict__ Gi, const float *__restrict__ df,
                                                           float *__restrict__ part) {
    using V = typename MM16<S>::vec;
    __shared__ __align__(16) unsigned char sT[2][kWBuf];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row = lane & 15, kk = lane >> 4;
    // waves s and s + 4 share a SIMD: half a tile apart, so that of a tile on
    // the diagonal, whose lower half is idle, each SIMD has a working wave
    const int wr = wave >> 2, we = (wave + 2 * wr) & 3;
    int te, tr, split, k;
    wide_block(P, te, tr, split, k);
    const int e0 = te * kWE, r0 = tr * kWR;
    if (P.dmin >= 32 && max_circ_dist(P.m, e0, kWE, r0, kWR) < P.dmin) return;
    const bool idle = e0 + 64 * we >= r0 + 64 * (wr + 1) ||
                      (P.dmin >= 32 && max_circ_dist(P.m, e0 + 64 * we, 64, r0 + 64 * wr, 64) < P.dmin);
    const int64_t N = P.N;
    const int64_t ks = (int64_t)split * P.kchunk;
    const int64_t ke = std::min<int64_t>(N, ks + P.kchunk);
    const int last = (int)((ke - ks + kF16KC - 1) / kF16KC) - 1;   // last chunk
    // staging: pixels p8 .. p8 + 7 of e rows r4, r4 + 128 and r row r4.  Rows at
    // or beyond m read row m - 1: their outputs are never read.
    const int sch = tid & 3, p8 = sch * 8, r4 = tid >> 2;
    const unsigned short *rowp[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const int r = std::min((j < 2 ? e0 + 128 * j : r0) + r4, P.m - 1);
        rowp[j] = reinterpret_cast<const unsigned short *>(Gr) + ((int64_t)k * P.m + r) * N;
    }
    const int64_t im = reinterpret_cast<const unsigned short *>(Gi) - reinterpret_cast<const unsigned short *>(Gr);
    u32x4 v[3][2];
    f4 d0, d1;
    auto load = [&](int c) {
        const int64_t xc = ks + (int64_t)c * kF16KC + p8;
        if (xc - p8 + kF16KC <= N) {   // workgroup-uniform
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                v[j][0] = *reinterpret_cast<const u32x4_a2 *>(rowp[j] + xc);
                v[j][1] = *reinterpret_cast<const u32x4_a2 *>(rowp[j] + im + xc);
            }
        } else {
            // the last chunk of the row: zero beyond N
#pragma unroll
            for (int j = 0; j < 3; ++j)
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const unsigned short *g = rowp[j] + a * im;
                        const unsigned lo = xc + 2 * q < N ? g[xc + 2 * q] : 0;
                        const unsigned hi = xc + 2 * q + 1 < N ? g[xc + 2 * q + 1] : 0;
                        v[j][a][q] = lo | (hi << 16);
                    }
        }
        d0 = *reinterpret_cast<const f4 *>(df + xc);   // zero beyond N
        d1 = *reinterpret_cast<const f4 *>(df + xc + 4);
    };
    auto store = [&](unsigned char *buf) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int a = 0; a < 2; ++a)
                *reinterpret_cast<u32x4 *>(buf + a * kWArrE + f16_off(r4 + 128 * j, sch)) = v[j][a];
#pragma unroll
        for (int a = 0; a < 2; ++a)
            *reinterpret_cast<u32x4 *>(buf + 2 * kWArrE + a * kWArrR + f16_off(r4, sch)) =
                f16_scale<S, V>(v[2][a], d0, d1);
    };
    f4 re[4][4], imv[4][4];
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int c = 0; c < 4; ++c) re[b][c] = imv[b][c] = f4{0, 0, 0, 0};
    auto mma = [&](const unsigned char *sa) {
        const unsigned char *sb = sa + 2 * kWArrE;
        V b_r[4], b_i[4];
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
            const int o = f16_off(64 * wr + 16 * cb + row, kk);
            b_r[cb] = *reinterpret_cast<const V *>(sb + o);
            b_i[cb] = *reinterpret_cast<const V *>(sb + kWArrR + o);
        }
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int o = f16_off(64 * we + 16 * b + row, kk);
            const V a_r = *reinterpret_cast<const V *>(sa + o);
            const V a_i = *reinterpret_cast<const V *>(sa + kWArrE + o);
            const V a_n = neg(a_i);
            // (ar + i ai)(br + i bi) = ar br - ai bi + i (ar bi + ai br)
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) {
                re[b][cb] = MM16<S>::mma(a_r, b_r[cb], re[b][cb]);
                imv[b][cb] = MM16<S>::mma(a_r, b_i[cb], imv[b][cb]);
            }
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) {
                re[b][cb] = MM16<S>::mma(a_n, b_i[cb], re[b][cb]);
                imv[b][cb] = MM16<S>::mma(a_i, b_r[cb], imv[b][cb]);
            }
        }
    };
    load(0);
    store(sT[0]);
    load(std::min(1, last));
    auto kloop = [&](auto first) {   // first: convert before multiplying
        for (int c = 0; c <= last; ++c) {
            lds_barrier();   // chunk c is in LDS, and no wave still reads the other buffer
            unsigned char *sn = sT[(c & 1) ^ 1];
            // (the last two steps convert and load the last chunk again, unused)
            if (decltype(first)::value) {
                store(sn);
                load(std::min(c + 2, last));
                __builtin_amdgcn_sched_barrier(0);
            }
            if (!idle) mma(sT[c & 1]);
            if (!decltype(first)::value) {
                __builtin_amdgcn_sched_barrier(0);
                store(sn);
                load(std::min(c + 2, last));
            }
        }
    };
    if (wr == 0)
        kloop(std::true_type());
    else
        kloop(std::false_type());
    if (idle) return;
    float *pp = part + ((int64_t)split * P.nf + k) * P.mp * P.mp * 2;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
            const int r = r0 + 64 * wr + 16 * cb + row;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int ee = e0 + 64 * we + 16 * b + 4 * kk + i;
                *reinterpret_cast<f2 *>(pp + ((int64_t)ee * P.mp + r) * 2) = f2{re[b][cb][i], imv[b][cb][i]};
            }
        }
    }
}

// The same tile for rows of whole 16-byte pieces, in pieces of 128 bytes (L2
// serves about as many requests of 128 bytes a second as of 64).  The e rows of
// 64 pixels go straight to LDS, a pair of steps ahead, into two buffers of 64
// KB; the r rows pass through registers, loaded a pair ahead, multiplied by
// delta and stored one step's half at a time.  Piece c of an e row is at
// position c ^ (row / 2 mod 8), so that the 16 rows of a fragment lie on
// distinct banks.  Pieces beyond the table's last pixel come from the zeros
// after delta.  BF16, 1024 elements / 1100^2, four frequencies: 34.9 (pieces of
// 64 bytes, k_forward16_wide) -> 22.6 ms, 0.90 PFLOP/s, near the 1.0 to 1.1 at
// which the card's power limits its clock; 1024 / 480^2, one, 1.19 -> 0.99 ms.
// (Direct loads of the e rows one step later, behind the conversion of the r
// rows, so that it need not wait for them: 23.7 ms.)
constexpr int kDArrE = kWE * 128;   // one array of the e side (bytes)
typedef __attribute__((address_space(3))) void lds_void_t;
template <int I>
using Idx = std::integral_constant<int, I>;

template <typename S>
__global__ void __launch_bounds__(512, 2) k_forward16_direct(FwdParams P, const S *__restrict__ Gr,
                                                             const S *__restrict__ Gi, const float *__restrict__ df,
                                                             float *__restrict__ part) {
    using V = typename MM16<S>::vec;
    // separate objects, so that a direct load into one is known not to write
    // the one being read
    __shared__ __align__(16) unsigned char sE0[2 * kDArrE];
    __shared__ __align__(16) unsigned char sE1[2 * kDArrE];
    __shared__ __align__(16) unsigned char sR0[2 * kWArrR];
    __shared__ __align__(16) unsigned char sR1[2 * kWArrR];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row = lane & 15, kk = lane >> 4;
    // (waves and SIMDs, tiles and splits: as k_forward16_wide)
    const int wr = wave >> 2, we = (wave + 2 * wr) & 3;
    int te, tr, split, k;
    wide_block(P, te, tr, split, k);
    const int e0 = te * kWE, r0 = tr * kWR;
    if (P.dmin >= 32 && max_circ_dist(P.m, e0, kWE, r0, kWR) < P.dmin) return;
    const bool idle = e0 + 64 * we >= r0 + 64 * (wr + 1) ||
                      (P.dmin >= 32 && max_circ_dist(P.m, e0 + 64 * we, 64, r0 + 64 * wr, 64) < P.dmin);
    const int64_t N = P.N;
    const int64_t ks = (int64_t)split * P.kchunk;
    const int64_t ke = std::min<int64_t>(N, ks + P.kchunk);
    const int last = (int)((ke - ks + kF16KC - 1) / kF16KC) - 1;   // last step
    const int lastp = last >> 1;                                   // last pair of steps
    const unsigned short *gr = reinterpret_cast<const unsigned short *>(Gr) + (int64_t)k * P.m * N;
    const unsigned short *gi = reinterpret_cast<const unsigned short *>(Gi) + (int64_t)k * P.m * N;
    const unsigned short *zeros = reinterpret_cast<const unsigned short *>(df + N);
    // e side: wave w fills rows 64 (w mod 4) .. + 63 of array w / 4, eight rows an
    // instruction; r side: piece tid % 8 of rows tid / 8 and tid / 8 + 64.  Rows
    // at or beyond m read row m - 1: their outputs are never read.
    const unsigned short *ge = wave >> 2 ? gi : gr;
    const int l8 = lane >> 3;
    unsigned eoff[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int r = std::min(e0 + 64 * (wave & 3) + 8 * j + l8, P.m - 1) - std::min(e0, P.m - 1);
        eoff[j] = (unsigned)r * (unsigned)N + 8u * ((lane & 7) ^ ((4 * j + (l8 >> 1)) & 7));
    }
    ge += (int64_t)std::min(e0, P.m - 1) * N;
    const int half = (tid >> 2) & 1, sch = tid & 3, p8 = 8 * (tid & 7), r8 = tid >> 3;
    unsigned roff[2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
        roff[j] = (unsigned)(std::min(r0 + r8 + 64 * j, P.m - 1) - std::min(r0, P.m - 1)) * (unsigned)N + (unsigned)p8;
    const int64_t rbase = (int64_t)std::min(r0, P.m - 1) * N;
    auto load_e = [&](int p, unsigned char *buf) {
        const int64_t x0 = ks + 64 * (int64_t)p;
        unsigned char *d = buf + (wave >> 2) * kDArrE + 64 * (wave & 3) * 128;
        const unsigned short *g = ge + x0;
        const int left = (int)std::min<int64_t>(N - x0, 64);   // pixels of the table (no branch: see step)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int px = 8 * ((lane & 7) ^ ((4 * j + (l8 >> 1)) & 7));
            __builtin_amdgcn_global_load_lds(px < left ? g + eoff[j] : zeros, (lds_void_t *)(d + j * 1024), 16, 0, 0);
        }
    };
    u32x4 v[2][2];
    f4 d0, d1;
    auto load_r = [&](int p) {
        const int64_t x0 = ks + 64 * (int64_t)p;
        const unsigned short *ga = gr + rbase + x0, *gb = gi + rbase + x0;
        const bool in = x0 + p8 < N;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            v[j][0] = *reinterpret_cast<const u32x4 *>(in ? ga + roff[j] : zeros);
            v[j][1] = *reinterpret_cast<const u32x4 *>(in ? gb + roff[j] : zeros);
        }
        const float *q = df + (in ? x0 + p8 : N);
        d0 = *reinterpret_cast<const f4 *>(q);
        d1 = *reinterpret_cast<const f4 *>(q + 4);
    };
    auto convert = [&]() {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int a = 0; a < 2; ++a) v[j][a] = f16_scale<S, V>(v[j][a], d0, d1);
    };
    auto store_r = [&](int h, unsigned char *buf) {
        if (half != h) return;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int a = 0; a < 2; ++a)
                *reinterpret_cast<u32x4 *>(buf + a * kWArrR + f16_off(r8 + 64 * j, sch)) = v[j][a];
    };
    f4 re[4][4], imv[4][4];
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int c = 0; c < 4; ++c) re[b][c] = imv[b][c] = f4{0, 0, 0, 0};
    const int te0 = (64 * we + row) * 128 + 16 * (kk ^ ((row >> 1) & 7));
    const int tr0 = f16_off(64 * wr + row, kk);
    auto mma = [&](const unsigned char *sa, int h, const unsigned char *sb) {
        V b_r[4], b_i[4];
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
            b_r[cb] = *reinterpret_cast<const V *>(sb + tr0 + 16 * cb * 64);
            b_i[cb] = *reinterpret_cast<const V *>(sb + kWArrR + tr0 + 16 * cb * 64);
        }
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int o = (te0 ^ (64 * h)) + 16 * b * 128;
            const V a_r = *reinterpret_cast<const V *>(sa + o);
            const V a_i = *reinterpret_cast<const V *>(sa + kDArrE + o);
            const V a_n = neg(a_i);
            // (ar + i ai)(br + i bi) = ar br - ai bi + i (ar bi + ai br)
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) {
                re[b][cb] = MM16<S>::mma(a_r, b_r[cb], re[b][cb]);
                imv[b][cb] = MM16<S>::mma(a_r, b_i[cb], imv[b][cb]);
            }
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) {
                re[b][cb] = MM16<S>::mma(a_n, b_i[cb], re[b][cb]);
                imv[b][cb] = MM16<S>::mma(a_i, b_r[cb], imv[b][cb]);
            }
        }
    };
    // step c (I = c mod 4; pair c / 2, half c mod 2).  Even steps store the
    // second half of their pair's r rows and issue the next pair's loads; odd
    // ones convert those r rows and store their first half.  (The last steps
    // load and store the last pair again, unused.)
    auto step = [&](int c, auto itag, auto first) {
        constexpr int I = decltype(itag)::value, H = I & 1;
        unsigned char *se = I & 2 ? sE1 : sE0, *sn = I & 2 ? sE0 : sE1;
        if (!H) __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));   // this pair's e rows
        lds_barrier();   // step c is in LDS, and no wave still reads the other buffers
        auto stage = [&]() {
            if (H) {
                convert();
                store_r(0, sR0);
            } else {
                store_r(1, sR1);
                const int p = std::min((c >> 1) + 1, lastp);
                load_r(p);
                __builtin_amdgcn_sched_barrier(0);
                load_e(p, sn);
            }
        };
        if (decltype(first)::value) {
            stage();
            __builtin_amdgcn_sched_barrier(0);
        }
        if (!idle) mma(se, H, H ? sR1 : sR0);
        if (!decltype(first)::value) {
            __builtin_amdgcn_sched_barrier(0);
            stage();
        }
    };
    load_e(0, sE0);
    load_r(0);
    convert();
    store_r(0, sR0);
    auto kloop = [&](auto first) {   // first: stage before multiplying
        for (int c = 0; c <= last; c += 4) {
            step(c, Idx<0>(), first);
            if (c + 1 <= last) step(c + 1, Idx<1>(), first);
            if (c + 2 <= last) step(c + 2, Idx<2>(), first);
            if (c + 3 <= last) step(c + 3, Idx<3>(), first);
        }
    };
    if (wr == 0)
        kloop(std::true_type());
    else
        kloop(std::false_type());
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));   // no direct load outlives the workgroup's LDS
    if (idle) return;
    float *pp = part + ((int64_t)split * P.nf + k) * P.mp * P.mp * 2;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
            const int r = r0 + 64 * wr + 16 * cb + row;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int ee = e0 + 64 * we + 16 * b + 4 * kk + i;
                *reinterpret_cast<f2 *>(pp + ((int64_t)ee * P.mp + r) * 2) = f2{re[b][cb][i], imv[b][cb][i]};
            }
        }
    }
}

}  // namespace

// ---------------------------------------------------------------- host side
// Compute units of the current device (256 on MI355X), queried on every
// call: the library keeps no mutable state between calls.
static int device_cus() {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
        return 256;
    return cus;
}

// Wide tiles by direct loads: rows of whole 16-byte pieces, 256 N elements
// within 32-bit offsets.
static bool fwd16_direct(int64_t N) { return N % 8 == 0 && N < ((int64_t)1 << 23); }

// The wide-tile 16-bit kernel: rows that are not 16-byte aligned, which the 64
// x 64-tile kernel reads element by element (us per call, that / this: 64
// elements / 255x301 107 / 153, 96 200 / 151, 200 548 / 171, 1024 8906 /
// 1214), and aligned rows of large problems, where the small tiles are bound by
// the bytes they move, unless padding to 256 rows costs more: that / this with
// direct loads 512 / 128^2 58 / 59, 1024 / 200^2, two frequencies, 603 / 457,
// 600 / 480^2 601 / 655, 1024 / 1100^2, four, 67.8 / 22.6 ms; more padding pays
// from about 10^6 pixels on: 256 / 728^2 293 / 358, 384 / 728^2 657 / 690, 256 /
// 1100^2 979 / 652, 384 / 1000^2 1686 / 1297, 300 / 480^2 186 / 347.
static bool fwd16_wide(const rb_geometry *g, rb_dtype dt) {
    if (dt != RB_BF16 && dt != RB_F16) return false;
    const int64_t N = (int64_t)g->nx * g->ny;
    if (N % 8 != 0) return g->m > 64;
    const int mp = (g->m + kWE - 1) / kWE * kWE;
    return (g->m >= 512 && N >= 32768 && 5 * mp <= 6 * g->m) || (g->m >= 256 && fwd16_direct(N) && N >= kWidePx &&
                                                                2 * mp <= 3 * g->m);
}

// FP32 tables on the FP16 cores: rings that fill more than half of a 128-element
// tile, and grids whose sums are long enough for its accuracy and, with small rings,
// for its two more launches.  us per call on the FP32 cores / split, two
// frequencies: 64 elements / 480^2 127 / 159; 96 / 64x66 25 / 26, 96 / 128^2 44 / 35,
// 96 / 480^2 297 / 170, 97 / 301x255 234 / 69; 256 / 64x66 48 / 41, 256 / 128^2 101 / 66,
// 256 / 255x301 925 / 229; 512 / 64x66 105 / 64; 1024 / 480^2 12270 / 6610.  At 512 / 32^2 it
// would be 48 / 41, but with splits of 16 pixels the FP32 cores are nearer to
// FP64 there (relative L2 error at 257 to 1000 elements, split against ordered pairs on
// the FP32 cores: 16^2 up to 1.24 of it, 32^2 1.11; from 48^2 on below it).
static bool fwd32_split(const rb_geometry *g, rb_dtype dt) {
    return dt == RB_F32 && g->m > 64 && (int64_t)g->nx * g->ny >= (g->m > 256 ? 4096 : 8192);
}

// The FP32 kernel with direct loads: rows of whole 16-byte chunks.
static bool fwd32_direct(const rb_geometry *g, rb_dtype dt) {
    return dt == RB_F32 && ((int64_t)g->nx * g->ny) % 4 == 0;
}

static FwdParams fwd_params(const rb_geometry *g, const double *freqs, int nf, rb_dtype dt) {
    FwdParams P;
    const bool fs = fwd32_split(g, dt);
    const bool wide = fwd16_wide(g, dt);
    const int tile = fs ? kFsT : (wide ? kWE : 64);
    P.m = g->m;
    P.mp = (g->m + tile - 1) / tile * tile;
    P.N = (int64_t)g->nx * g->ny;
    P.nf = nf;
    P.ntl = P.mp / (wide ? kWR : tile);
    // tiles on or above the diagonal (the wide ones: ntl - 2 te in row te)
    const int ntri = wide ? P.ntl / 2 * (P.ntl / 2 + 1) : P.ntl * (P.ntl + 1) / 2;
    // about four rounds of resident workgroups (two per CU, four for the
    // FP32 kernel with direct loads), rounded down so the last round is full;
    // but no split is shorter than kMinSplitPx, and with the large tiles and 16-bit
    // rows of whole 16-byte pieces, beyond one round, than kFewSplitPx pixels: a
    // split's partial sums (a tile of them, written and read once) cost as much as some
    // tens of pixels (BF16, without / with: 97 elements / 230x152, three frequencies,
    // 42.9 / 33.2 us, 256 / 128^2, two, 44.0 / 35.4, 768 / 64x66, two, 60.1 / 56.2).  The
    // other small tiles need the waves: 256 elements / 128^2 FP64 245 us, with the longer
    // splits 304; 40 / 655x501, rows not aligned, BF16 235 and 280.
    //
    // The FP32 cores' kernels add to a split's sums once per four pixels; with splits of
    // 64 or 512 pixels in FP32 the error of the result is up to 2.9 times that with 16 (20
    // elements / 41x82, two frequencies: 3.3e-8, 9.1e-8).  Where splits of 16 to 64 pixels
    // would come out (sum64; rows of whole 16-byte pieces), the sums of 16 pixels are
    // added in FP64 within a split instead, and the splits are few: us per call, FP32
    // partials of 16 pixels and so, 33 elements / 266x194, one frequency, 66 / 32, 64 /
    // 128^2, two, 34 / 25, 200 / 80^2, two, 54 / 48; longer splits gain nothing by it (64 /
    // 480^2, two, 130 / 135, 1000 / 32^2, two, 99 / 119, 64 / 1100^2, four, 926 / 1199).
    // Rows that are not aligned keep splits of 16 pixels.
    P.sum64 = !fs && fwd32_direct(g, dt) && P.N <= 64 * (int64_t)(16 * device_cus() / (ntri * nf));
    const int resident = (fs || wide ? 1 : (fwd32_direct(g, dt) && !P.sum64 ? 4 : 2)) * device_cus();
    int64_t most = dt == RB_F32 && !fs ? (P.N + kMinSplitPx32 - 1) / kMinSplitPx32 : P.N / kMinSplitPx;
    const bool small16 = (dt == RB_BF16 || dt == RB_F16) && !wide;
    if (P.sum64) most = (P.N + kMinSplitPx - 1) / kMinSplitPx;
    if (fs || wide || P.sum64 || (small16 && P.N % 8 == 0))
        most = std::max<int64_t>(P.N / kFewSplitPx, std::min<int64_t>(most, resident / (ntri * nf)));
    if (dt == RB_F64)   // within one round, a step each (16 elements / 32^2: 16.6 -> 11.6 us)
        most = std::max<int64_t>(most, std::min<int64_t>((P.N + 15) / 16, resident / (ntri * nf)));
    int nsplit = std::max<int64_t>(1, std::min<int64_t>(4 * resident / (ntri * nf), most));
    // whole rounds where that is less work in a row (rounds / splits): a last
    // round with a tenth of the workgroups takes as long as a full one.  us,
    // before and now: 97 elements / 301x255, two frequencies, FP32 113 / 77 (1.1
    // rounds -> 1), BF16 152 / 119, 256 / 301x255 FP32 246 / 216, BF16 190 / 149
    const int64_t full = (int64_t)nsplit * ntri * nf / resident * resident / (ntri * nf);
    auto rounds = [&](int64_t n) { return (n * ntri * nf + resident - 1) / resident; };
    if ((dt != RB_F32 || fs || P.sum64) && full > 0 && rounds(full) * nsplit < rounds(nsplit) * full) nsplit = (int)full;
    // the kernels with direct loads (FP32, and 16-bit for large rings) also
    // keep a split to at most kFdSplitPx pixels: the tiles of a split share
    // its table rows in L2 only while they stay within a few k-steps of each
    // other, and long workgroups drift apart (FP32, 1024 elements / 1100^2:
    // 7 splits 144.4 ms, 30 splits 138.1 ms, 60 splits 135.0 ms for the
    // public call)
    if (fs || fwd32_direct(g, dt) || wide)
        nsplit = std::max<int64_t>(nsplit, (P.N + kFdSplitPx - 1) / kFdSplitPx);
    const int kq = (fs || dt == RB_BF16 || dt == RB_F16) ? 32 : 16;
    int64_t kchunk = (P.N + nsplit - 1) / nsplit;
    kchunk = (kchunk + kq - 1) / kq * kq;
    if (kchunk < kq) kchunk = kq;
    nsplit = (int)((P.N + kchunk - 1) / kchunk);
    P.nsplit = nsplit;
    P.kchunk = kchunk;
    P.ntri = ntri;
    P.dmin = 0;
    const double dA = g->h * g->h;
    for (int k = 0; k < nf; ++k) {
        const double om = 2.0 * M_PI * (freqs ? freqs[k] : 1.0);
        P.cg[k] = om * om * dA;
    }
    return P;
}

// workspace: max |delta|, the split partials, delta as float
struct FwdWs {
    double *dmax, *dparts;
    void *part;
    float *df;
    // k_forward_split: row scales, |delta| maxima, delta's scale, list, flags
    float *fscale, *fpart, *fdscale;
    int *redo;
    uint8_t *flags;
    int64_t nflags;
};

static FwdWs carve_fwd(Carver &c, const FwdParams &P, rb_dtype dt, bool fs) {
    const size_t es = dt == RB_F64 || P.sum64 ? 8 : 4;
    FwdWs w;
    w.dmax = c.take<double>(1);
    w.dparts = (dt == RB_BF16 || dt == RB_F16) ? c.take<double>(kReduceBlocks) : nullptr;
    w.part = c.take<char>((size_t)P.nsplit * P.nf * P.mp * P.mp * 2 * es);
    w.df = (fs || dt == RB_BF16 || dt == RB_F16 || (dt == RB_F32 && P.N % 4 == 0)) ? c.take<float>((size_t)P.N + 32)
                                                                                     : nullptr;
    w.nflags = fs ? (int64_t)P.nf * P.nsplit * P.ntl : 0;
    if (fs) {
        w.fscale = c.take<float>((size_t)P.nf * P.m);
        w.fpart = c.take<float>(kReduceBlocks);
        w.fdscale = c.take<float>(1);
        w.redo = c.take<int>((size_t)w.nflags + 1);
        w.flags = c.take<uint8_t>((size_t)w.nflags);
    }
    return w;
}

size_t forward_workspace_bytes(const rb_geometry *g, int nf, rb_dtype dt) {
    FwdParams P = fwd_params(g, nullptr, nf, dt);
    Carver c(nullptr, 0);
    carve_fwd(c, P, dt, fwd32_split(g, dt));
    return c.used + 256;
}

rb_status forward_impl(const rb_geometry *g, const void *G_re, const void *G_im, const float *gscale,
                       rb_dtype dt, const double *freqs, int nf, const double *delta, double *d_out, void *ws,
                       size_t ws_bytes, hipStream_t st, int dmin) {
    if (ws_bytes < forward_workspace_bytes(g, nf, dt)) {
        set_error("forward workspace too small: need %zu bytes", forward_workspace_bytes(g, nf, dt));
        return RB_ENOMEM;
    }
    FwdParams P = fwd_params(g, freqs, nf, dt);
    P.dmin = dmin;
    Carver c(ws, ws_bytes);
    const bool fs = fwd32_split(g, dt);
    FwdWs w = carve_fwd(c, P, dt, fs);
    FwdSplitOut so{nullptr, nullptr, nullptr, kFsT};
    const unsigned nblk = (unsigned)((int64_t)P.ntri * P.nsplit * nf);
    auto reduce = [&](auto tag, const float *gs, const double *dmax) {
        using T = decltype(tag);
        if ((int64_t)nf * P.m * P.m >= kRedEntries)
            k_forward_reduce<T, 1, 64>
                <<<dim3(blocks_for(P.m, 64), P.m, nf), 64, 0, st>>>(P, (const T *)w.part, gs, dmax, d_out, so);
        else
            k_forward_reduce<T, 8, 256>
                <<<dim3(blocks_for(P.m, 32), P.m, nf), 256, 0, st>>>(P, (const T *)w.part, gs, dmax, d_out, so);
    };
    switch (dt) {
        case RB_F64: {
            dim3 grid(P.ntri, P.nsplit, nf);
            k_forward_f64<<<grid, 256, 0, st>>>(P, (const double *)G_re, (const double *)G_im, delta,
                                                (double *)w.part);
            RB_LAUNCHED();
            reduce(double(), nullptr, nullptr);
            break;
        }
        case RB_F32:
            if (fs) {
                const float *gr = (const float *)G_re, *gi = (const float *)G_im;
                float *pt = (float *)w.part;
                k_fs_scales<<<nf * P.m + kReduceBlocks, 256, 0, st>>>(P.N, nf * P.m, gr, gi, delta, w.fscale,
                                                                      w.fpart);
                RB_LAUNCHED();
                k_fs_delta<<<blocks_for(P.N + 32, 256), 256, 0, st>>>(P.N, P.N + 32, delta, w.fpart, w.df, w.fdscale,
                                                                      nf * P.m, w.fscale, w.redo, w.flags, w.nflags);
                RB_LAUNCHED();
                const unsigned nl = (unsigned)std::min<int64_t>(4 * P.ntl * w.nflags, (P.N % 4 == 0 ? 4 : 2) * device_cus());
                k_forward_split<<<nblk, 512, 0, st>>>(P, gr, gi, w.df, w.fscale, pt, w.redo, w.flags);
                RB_LAUNCHED();
                if (P.N % 4 == 0)
                    k_forward_f32_list<true><<<nl, 256, 0, st>>>(P, gr, gi, w.df, pt, w.redo, w.flags);
                else
                    k_forward_f32_list<false><<<nl, 256, 0, st>>>(P, gr, gi, w.df, pt, w.redo, w.flags);
                so = FwdSplitOut{w.flags, w.fscale, w.fdscale, kFsT};
            } else if (fwd32_direct(g, dt)) {
                k_delta_cast<<<blocks_for(P.N + 16, 256), 256, 0, st>>>(P.N, P.N + 16, delta, w.df);
                RB_LAUNCHED();
                const float *gr = (const float *)G_re, *gi = (const float *)G_im;
                if (P.sum64) {
                    k_forward_f32<double><<<nblk, 256, 0, st>>>(P, gr, gi, w.df, (double *)w.part);
                    RB_LAUNCHED();
                    reduce(double(), gscale, nullptr);
                    break;
                }
                k_forward_f32<float><<<nblk, 256, 0, st>>>(P, gr, gi, w.df, (float *)w.part);
            } else {
                k_forward_f32_regs<<<dim3(P.ntri, P.nsplit, nf), 256, 0, st>>>(P, (const float *)G_re,
                                                                               (const float *)G_im, delta,
                                                                               (float *)w.part);
            }
            RB_LAUNCHED();
            reduce(float(), gscale, nullptr);
            break;
        case RB_BF16:
        case RB_F16:
            RB_TRY(reduce_absmax_f64(delta, P.N, w.dparts, w.dmax, st));
            k_delta_f32<<<blocks_for(P.N + 32, 256), 256, 0, st>>>(P.N, P.N + 32, delta, w.dmax, w.df);
            RB_LAUNCHED();
            if (fwd16_wide(g, dt)) {
                if (fwd16_direct(P.N)) {
                    if (dt == RB_BF16)
                        k_forward16_direct<<<nblk, 512, 0, st>>>(P, (const __hip_bfloat16 *)G_re,
                                                                 (const __hip_bfloat16 *)G_im, w.df,
                                                                 (float *)w.part);
                    else
                        k_forward16_direct<<<nblk, 512, 0, st>>>(P, (const __half *)G_re, (const __half *)G_im, w.df,
                                                                 (float *)w.part);
                } else if (dt == RB_BF16)
                    k_forward16_wide<<<nblk, 512, 0, st>>>(P, (const __hip_bfloat16 *)G_re,
                                                           (const __hip_bfloat16 *)G_im, w.df, (float *)w.part);
                else
                    k_forward16_wide<<<nblk, 512, 0, st>>>(P, (const __half *)G_re, (const __half *)G_im, w.df,
                                                           (float *)w.part);
            } else if (dt == RB_BF16)
                k_forward16_lds<__hip_bfloat16><<<nblk, 256, 0, st>>>(P, (const __hip_bfloat16 *)G_re,
                                                                      (const __hip_bfloat16 *)G_im, w.df,
                                                                      (float *)w.part);
            else
                k_forward16_lds<__half><<<nblk, 256, 0, st>>>(P, (const __half *)G_re, (const __half *)G_im,
                                                              w.df, (float *)w.part);
            RB_LAUNCHED();
            reduce(float(), gscale, w.dmax);
            break;
    }
    RB_LAUNCHED();
    return RB_OK;
}

rb_status check_contraction(const rb_geometry *g, const void *G_re, const void *G_im, const float *scale,
                                   rb_dtype dt, const double *freqs, int32_t nf) {
    RB_TRY(check_geometry(g));
    RB_TRY(check_freqs(freqs, nf));
    RB_CHECK_ARG(dt >= RB_F64 && dt <= RB_F16, "unknown dtype %d", (int)dt);
    RB_CHECK_ARG(G_re && G_im, "G_re/G_im are NULL");
    RB_CHECK_ARG(((uintptr_t)G_re & 15) == 0 && ((uintptr_t)G_im & 15) == 0,
                 "G_re/G_im must be 16-byte aligned (the kernels read rows in 16-byte pieces)");
    RB_CHECK_ARG(!(dt == RB_BF16 || dt == RB_F16) || scale, "scale is required for 16-bit storage");
    return RB_OK;
}

}  // namespace rb

extern "C" {

size_t rb_forward_workspace_bytes(const rb_geometry *g, int32_t nf, rb_dtype dtype) {
    if (rb::check_geometry(g) != RB_OK || nf < 1 || nf > RB_MAX_NF) return 0;
    return rb::forward_workspace_bytes(g, nf, dtype);
}

rb_status rb_born_forward(const rb_geometry *g, const void *G_re, const void *G_im, const float *scale,
                          rb_dtype dtype, const double *freqs_hz, int32_t nf, const double *delta, double *d_out,
                          void *ws, size_t ws_bytes, void *stream) {
    rb::clear_error();
    RB_TRY(rb::check_contraction(g, G_re, G_im, scale, dtype, freqs_hz, nf));
    RB_CHECK_ARG(delta && d_out, "delta/d_out are NULL");
    RB_CHECK_ARG(ws, "workspace is NULL");
    return rb::forward_impl(g, G_re, G_im, scale, dtype, freqs_hz, nf, delta, d_out, ws, ws_bytes,
                            rb::as_stream(stream));
}

}  // extern "C"
