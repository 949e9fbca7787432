// Weighted adjoint (backprojection) of the Born operator with the diagonal of
// the Gauss-Newton Hessian (paper, Inverse Problem section, Eqs. 8-10;
// linearisation of Eq. 1 in q = 1/c^2 with Green's functions from Eqs. 4-5).
//
//   grad(x) = omega^2 h^2 Re sum_e conj(G_e(x)) Y_e(x),
//   Y_e(x)  = sum_r A_er conj(G_r(x)),      A = W . D
//   hd(x)   = omega^4 h^4 sum_e |G_e(x)|^2 Z_e(x),
//   Z_e(x)  = sum_r W_er |G_r(x)|^2
//
// A dense contraction over emitter x receiver pairs, so it runs on the matrix
// cores.  The complex product is expanded into real MFMAs and the reduction
// over e against G_e(x) is fused into the epilogue, so Y and Z never leave
// registers.  A k-permutation (lane group kk supplies k = 4 kk + s at MFMA
// step s) lets each lane fetch its A fragment with one vector load.
//
// Both sums are symmetric in (e, r) apart from A and W, so each unordered
// pair is contracted once, with (A_er + A_re) / 2 and (W_er + W_re) / 2 and
// the factor 2 in the constants (k_adj_prep).  Of the two 32 x 32 blocks (I,
// J) and (J, I) the one whose J follows I by less than half the ring, in
// circular block order, is kept: every emitter block then has about half the
// ring's receiver blocks, whatever its place in the ring, and passes of
// consecutive emitter blocks share most of theirs.  Blocks that are not kept,
// and blocks whose weights are all zero (the receiver selection removes a
// band around the diagonal), are skipped: neither staged nor multiplied.
// Against contracting both orders (1024 elements / 1100^2, four frequencies;
// bound by the matrix cores): FP32 (on its own cores) 209.9 -> 105.6 ms, BF16
// 32.9 -> 17.2 ms; 256 / 480^2, three frequencies, FP32: 2.31 -> 1.46 ms (three
// or four chunks per pass are left, so a pass's fixed cost weighs more).
#include <algorithm>
#include <cmath>
#include <mutex>
#include <type_traits>

#include "born.h"
#include "common.h"
#include "mma.h"

namespace rb {
namespace {

// ------------------------------------------------------------------ FP64
// WG = 4 waves; wave w owns 16 CB pixels of one frequency and takes the
// emitters of its pass group, 16 RB at a time, against all their receivers.
// An FP64 MFMA runs 64 cycles, so the operands come straight from memory; what
// bounds the kernel is that every SIMD has a wave: a workgroup per (pixel
// tile, frequency), 64 pixels where 128 would leave compute units idle.  With
// a workgroup per 128 pixels over all frequencies and the Hessian product
// always formed, and now, two frequencies: 64 elements / 128^2 64 -> 37 us,
// 256 / 480^2 4.18 -> 2.65 ms (1.5 ms of MFMA time at 78.6 TFLOP/s).
template <typename T, int RB, int CB, bool HESS>
__global__ void __launch_bounds__(256) k_adjoint(AdjParams P, const T *__restrict__ Gr, const T *__restrict__ Gi,
                                                 const T *__restrict__ Ar, const T *__restrict__ Ai,
                                                 const T *__restrict__ Wt, const uint8_t *__restrict__ flags,
                                                 double *__restrict__ pg, double *__restrict__ ph) {
    using acc_t = typename MM<T>::acc;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int row = lane & 15, kk = lane >> 4;
    const int64_t N = P.N;
    const int64_t xw = (int64_t)blockIdx.x * (64 * CB) + (int64_t)wave * 16 * CB;
    const int k = blockIdx.y;
    const T *gr = Gr + (int64_t)k * P.m * N;
    const T *gi = Gi + (int64_t)k * P.m * N;
    const T *ar = Ar + (int64_t)k * P.mp * P.mp;
    const T *ai = Ai + (int64_t)k * P.mp * P.mp;
    const T *wt = Wt + (int64_t)k * P.mp * P.mp;
    const uint8_t *fl = flags + (int64_t)k * P.nb * P.nb;
    T gp[CB], hp[CB];
    int64_t xs[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) {
        gp[c] = hp[c] = T(0);
        xs[c] = min(xw + 16 * c + row, N - 1);   // pixels beyond N: the last one, dropped below
    }
    // (16 elements at a time: of a 32-element block only those below m)
    for (int ec = 0; ec < P.m; ec += 16 * RB) {
        acc_t yr[RB][CB], yn[RB][CB], z[RB][CB];
#pragma unroll
        for (int b = 0; b < RB; ++b)
#pragma unroll
            for (int c = 0; c < CB; ++c) yr[b][c] = yn[b][c] = z[b][c] = acc_t{0, 0, 0, 0};
        for (int rc = 0; rc < P.m; rc += 16) {
            bool on[RB];
            bool any = false;
#pragma unroll
            for (int b = 0; b < RB; ++b) {
                on[b] = ec + 16 * b < P.m && fl[(ec + 16 * b) / 32 * P.nb + rc / 32];
                any |= on[b];
            }
            if (!any) continue;
            T br[4][CB], bi[4][CB], b2[4][CB];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                // rows at or beyond m: the last one (their A and W are zero)
                const int64_t ro = (int64_t)min(rc + 4 * kk + s, P.m - 1) * N;
#pragma unroll
                for (int c = 0; c < CB; ++c) {
                    br[s][c] = gr[ro + xs[c]];
                    bi[s][c] = gi[ro + xs[c]];
                    if (HESS) b2[s][c] = br[s][c] * br[s][c] + bi[s][c] * bi[s][c];
                }
            }
#pragma unroll
            for (int b = 0; b < RB; ++b) {
                if (!on[b]) continue;
                const int64_t off = (int64_t)(ec + 16 * b + row) * P.mp + rc + 4 * kk;
                T va[4], vi[4], vw[4];
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    va[s] = ar[off + s];
                    vi[s] = ai[off + s];
                    if (HESS) vw[s] = wt[off + s];
                }
#pragma unroll
                for (int s = 0; s < 4; ++s) {
#pragma unroll
                    for (int c = 0; c < CB; ++c) {
                        yr[b][c] = MM<T>::mma(va[s], br[s][c], yr[b][c]);
                        yn[b][c] = MM<T>::mma(va[s], bi[s][c], yn[b][c]);
                    }
#pragma unroll
                    for (int c = 0; c < CB; ++c) {
                        yr[b][c] = MM<T>::mma(vi[s], bi[s][c], yr[b][c]);
                        yn[b][c] = MM<T>::mma(-vi[s], br[s][c], yn[b][c]);
                        if (HESS) z[b][c] = MM<T>::mma(vw[s], b2[s][c], z[b][c]);
                    }
                }
            }
        }
        // fused epilogue: reduce over the e rows of this chunk against G_e
        // (rows at or beyond m: the last one, whose Y and Z are zero)
#pragma unroll
        for (int b = 0; b < RB; ++b) {
            if (ec + 16 * b >= P.m) break;   // uniform
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int64_t eo = (int64_t)min(ec + 16 * b + MM<T>::out_row(kk, i), P.m - 1) * N;
#pragma unroll
                for (int c = 0; c < CB; ++c) {
                    const T ge_r = gr[eo + xs[c]], ge_i = gi[eo + xs[c]];
                    gp[c] += ge_r * yr[b][c][i] - ge_i * yn[b][c][i];
                    if (HESS) hp[c] += (ge_r * ge_r + ge_i * ge_i) * z[b][c][i];
                }
            }
        }
    }
    // sum the four lane groups that hold the same pixel (fixed order)
#pragma unroll
    for (int c = 0; c < CB; ++c) {
        double g = (double)gp[c] * P.cg[k], h = (double)hp[c] * P.ch[k];
        g += __shfl_xor(g, 16);
        h += __shfl_xor(h, 16);
        g += __shfl_xor(g, 32);
        h += __shfl_xor(h, 32);
        const int64_t x = xw + 16 * c + row;
        if (kk == 0 && x < N) {
            pg[(int64_t)k * N + x] = g;
            if (HESS) ph[(int64_t)k * N + x] = h;
        }
    }
}

template <typename T>
__device__ __forceinline__ T cvt(double v);
template <>
__device__ __forceinline__ double cvt<double>(double v) { return v; }
template <>
__device__ __forceinline__ float cvt<float>(double v) { return (float)v; }
template <>
__device__ __forceinline__ __hip_bfloat16 cvt<__hip_bfloat16>(double v) { return __float2bfloat16((float)v); }
template <>
__device__ __forceinline__ __half cvt<__half>(double v) { return __float2half((float)v); }

// The power of two that brings a value of magnitude `top` into [2^(e-1),
// 2^e) (1 for 0): exact to apply and to take back.
constexpr int kSplitTopA = 15, kSplitTopG = 10;
// The ranges in which two FP16 pieces hold FP32's bits (see k_adjoint_split).
constexpr float kSplitMinA = 0x1p-14f, kSplitMinG = 0x1p-2f, kSplitMax = 65504.0f;
constexpr float kSplitLoA = 0x1p12f;   // scale of the low pieces of A
__device__ __forceinline__ float split_scale(float top, int e) {
    if (!(top > 0.0f)) return 1.0f;
    int x;
    (void)frexpf(fminf(top, 3.0e38f), &x);
    return ldexpf(1.0f, min(max(e - x, -100), 100));
}

// Which of the blocks (I, J) and (J, I), I != J, of nb blocks around the ring
// is kept: the one whose J lies less than nb / 2 after I; at exactly nb / 2,
// the one with I < J.  Diagonal blocks are kept as they are.
__device__ __forceinline__ bool adj_kept(int I, int J, int nb) {
    const int d = J >= I ? J - I : J - I + nb;
    return 2 * d < nb || (2 * d == nb && I < J);
}

// max |W D| of every kept pair of blocks (as float bits; max is
// order-independent) folded into amax[k], which starts at zero.  One
// workgroup per 32 x 32 block and frequency.
__global__ void __launch_bounds__(256) k_adj_amax(int m, int nb, const double *__restrict__ d,
                                                  const double *__restrict__ w, unsigned *__restrict__ amax) {
    __shared__ float sm[4];
    const int k = blockIdx.y, I = blockIdx.x / nb, J = blockIdx.x - (blockIdx.x / nb) * nb;
    float v = 0.0f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int e = I * 32 + (threadIdx.x >> 5) + 8 * q, r = J * 32 + (threadIdx.x & 31);
        if (e < m && r < m) {
            const int64_t o = ((int64_t)k * m + e) * m + r;
            const double wv = w[o];
            v = fmaxf(v, (float)fmax(fabs(wv * d[2 * o]), fabs(wv * d[2 * o + 1])));
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        const float b = fmaxf(fmaxf(sm[0], sm[1]), fmaxf(sm[2], sm[3]));
        if (b > 0.0f) atomicMax(amax + k, __float_as_uint(b));
    }
}

// Operands of the adjoint in the storage type, [nf][mp][mp], one workgroup
// per 32 x 32 block (I, J) and frequency: half of A = W . D plus its
// transpose (re, im), and of W, in the kept blocks; half of A and W in the
// diagonal blocks; entries beyond m are zero.  The other blocks are left
// unwritten: flags[k][I][J], 1 for a kept block with a nonzero weight, keeps
// the contraction from reading them.  The transposed block passes through
// LDS so that both blocks are read along rows.  For 16-bit types A is
// divided by ascale[k] = max |W D| (1 if that is 0); W is 0/1-valued in the
// inversion and stored unscaled (the mean of two weights stays in range).
// Orders: LAYOUT 0: rows of mp; 1: the same with receiver 4 s + kk of every
// 32-column chunk at column 8 kk + s (the operand order of k_adjoint_f32); 2:
// the blocks one after the other, [I][J], each as the A fragments of its two
// 16-row halves (lane 16 kk + row holds columns 8 kk .. 8 kk + 7 of the row),
// so that a fragment is one contiguous 1 KB load.  With `shi` (FP32 only) A is
// also stored as two FP16 pieces of A split_scale(amax[k]), each [I][J][re,
// im] in fragments, and W, which only the Hessian diagonal needs, is not;
// bad[k] is set if a value but zero is too small for them.
//
// In 16 bits the mean of a pair is rounded once where the pair was twice: the
// squared error is the same where its two values are independent or equal, up to
// twice as large where they are close (residuals of reciprocal data with noise).
// A block whose squared errors add up to more than kLowRatio + kLowDoubt / sqrt(pairs)
// times those of the ordered pairs gets flag 3, if its J is odd or the ring's last,
// and the low-order parts of A, the means less their 16-bit values, lie in the place
// of the block (J, I), which is not kept.  The contraction adds those in k-steps of
// their own: with half of the blocks free of rounding errors the sum's is that of the
// ordered pairs again (relative error of the gradient, 256 elements, residual
// reciprocal but for 5 %, FP16: 0.30 2^-11, without these 0.41 2^-11, with both orders
// of a pair 0.31 2^-11).  BF16, gradient, both orders / folded / with such steps: 1024 /
// 1100^2, four frequencies, 32.4 / 16.8 / 22.8 ms, 256 / 480^2, three, 463 / 337 / 423 us.
// (Up to kAdjLowBlocks blocks: see adj_chunks_low.)
// A ratio of few pairs says little; the line is three or more standard deviations
// from that of independent values.  (At kLowRatio alone blocks at the edge of the
// selected band got the flag by chance: FP16, 880 / 268x134, four frequencies, 623 us,
// now 599.)
// Two blocks around the ring would gain no k-step by it (the pass stages both
// chunks anyway), so there both orders are kept, each as the diagonal blocks.
constexpr float kLowRatio = 1.3f, kLowDoubt = 4.0f;
constexpr int kAdjLowBlocks = 64;
template <typename T, bool SCALED, int LAYOUT = 0>
__global__ void __launch_bounds__(256) k_adj_prep(int m, int mp, const double *__restrict__ d,
                                                  const double *__restrict__ w, const float *__restrict__ ascale,
                                                  T *__restrict__ Ar, T *__restrict__ Ai, T *__restrict__ Wt,
                                                  uint8_t *__restrict__ flags, _Float16 *__restrict__ shi = nullptr,
                                                  _Float16 *__restrict__ slo = nullptr, int *__restrict__ bad = nullptr) {
    __shared__ double tr[32][33], ti[32][33], tw[32][33];
    const int nb = mp / 32;
    const int k = blockIdx.y, I = blockIdx.x / nb, J = blockIdx.x - (blockIdx.x / nb) * nb;
    uint8_t *fl = flags + ((int64_t)k * nb + I) * nb + J;
    const bool fold = I != J && !(SCALED && nb == 2);
    if (fold && !adj_kept(I, J, nb)) {   // workgroup-uniform
        if (threadIdx.x == 0) *fl = 0;
        return;
    }
    const int col = threadIdx.x & 31, row0 = threadIdx.x >> 5;
    // (indices clamped, not guarded, so that all 24 loads are in flight
    // together: 64 elements, two frequencies, 5.2 -> 3.9 us)
    double lw[2][4], lr[2][4], li[2][4];   // this block, the transposed one
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = (h ? J : I) * 32 + row0 + 8 * q, r = (h ? I : J) * 32 + col;
            const int64_t o = ((int64_t)k * m + min(e, m - 1)) * m + min(r, m - 1);
            lw[h][q] = w[o];
            lr[h][q] = d[2 * o];
            li[h][q] = d[2 * o + 1];
        }
    const float as = ascale ? ascale[k] : 0.0f;   // 0 when every weight is zero
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = row0 + 8 * q;
            const bool in = (h ? J : I) * 32 + i < m && (h ? I : J) * 32 + col < m;
            lr[h][q] = in ? lw[h][q] * lr[h][q] : 0.0;
            li[h][q] = in ? lw[h][q] * li[h][q] : 0.0;
            lw[h][q] = in ? lw[h][q] : 0.0;
            if (h) {
                tr[i][col] = lr[h][q];
                ti[i][col] = li[h][q];
                tw[i][col] = lw[h][q];
            }
        }
    __syncthreads();
    const double half = SCALED && as > 0.0f ? 0.5 / (double)as : 0.5;
    // (blocks with less than half of their rows or columns in the ring hold too
    // few pairs to tell)
    const bool split = SCALED && fold && ((J & 1) || J == nb - 1) && 32 * max(I, J) + 16 <= m &&
                       nb <= kAdjLowBlocks;
    float err = 0.0f, errp = 0.0f;   // squared errors: of twice the means less kLowRatio the pairs'; the pairs'
    int pairs = 0;                   // of the wave
    bool any = false;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int i = row0 + 8 * q;
        double re = lr[0][q], im = li[0][q], wv = lw[0][q];
        any |= wv != 0.0;
        if (fold) {
            any |= tw[col][i] != 0.0;
            re += tr[col][i];
            im += ti[col][i];
            wv += tw[col][i];
        }
        const int c = LAYOUT == 1 ? 8 * (col & 3) + (col >> 2) : col;
        const int64_t blk = ((int64_t)k * nb + I) * nb + J;
        const int fr = 512 * (i >> 4) + 8 * (16 * (col >> 3) + (i & 15)) + (col & 7);
        const int64_t o = LAYOUT == 2 ? 1024 * blk + fr : ((int64_t)k * mp + I * 32 + i) * mp + J * 32 + c;
        Ar[o] = cvt<T>(re * half);
        Ai[o] = cvt<T>(im * half);
        if (SCALED || !shi) Wt[o] = cvt<T>(wv * 0.5);
        if constexpr (SCALED) {
            if (split) {   // workgroup-uniform
                const int64_t lo = 1024 * (((int64_t)k * nb + J) * nb + I) + fr;
                auto part = [&](double a, double b, T *A) {   // the pair; its mean is at A[o]
                    auto off = [](float v) { return MM16<T>::to_f(cvt<T>((double)v)) - v; };
                    const float r = (float)((a + b) * half) - MM16<T>::to_f(A[o]);
                    const float e = off((float)(a * (2.0 * half))) + off((float)(b * (2.0 * half)));
                    err += 4.0f * r * r - kLowRatio * e * e;
                    errp += e * e;
                    A[lo] = cvt<T>((double)r);
                };
                part(lr[0][q], tr[col][i], Ar);
                part(li[0][q], ti[col][i], Ai);
                Wt[lo] = T(0.0f);
                pairs += __popcll(__ballot(wv != 0.0));
            }
        } else if (shi) {
            const float sa = split_scale(as, kSplitTopA);
            const float vr = (float)(re * half) * sa, vi = (float)(im * half) * sa;
            const _Float16 hr = (_Float16)vr, hi = (_Float16)vi;
            const int64_t q = 2048 * blk + fr;
            shi[q] = hr;
            shi[q + 1024] = hi;
            slo[q] = (_Float16)((vr - (float)hr) * kSplitLoA);
            slo[q + 1024] = (_Float16)((vi - (float)hi) * kSplitLoA);
            const float top = fmaxf(fabsf(vr), fabsf(vi));
            if (top > 0.0f && top < kSplitMinA) bad[k] = 1;
        }
    }
    __shared__ float se[4], sp[4];
    __shared__ int sn[4];
    if (split) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            err += __shfl_xor(err, o);
            errp += __shfl_xor(errp, o);
        }
        if ((threadIdx.x & 63) == 0) {
            se[threadIdx.x >> 6] = err;
            sp[threadIdx.x >> 6] = errp;
            sn[threadIdx.x >> 6] = pairs;
        }
    }
    const int on = __syncthreads_or(any);
    if (threadIdx.x == 0) {
        bool low = false;
        if (split) {
            const float n = (float)(sn[0] + sn[1] + sn[2] + sn[3]);
            low = ((se[0] + se[1]) + (se[2] + se[3])) * sqrtf(n) > kLowDoubt * ((sp[0] + sp[1]) + (sp[2] + sp[3]));
        }
        *fl = on ? (low ? 3 : 1) : 0;
    }
}

// The receiver chunks (32 receivers each, at most 128) an emitter pass works
// on, as wave-uniform bit masks.  Bit 2 t stands for chunk t and bit 2 t + 1
// for chunk t + half, half a ring further on, and the chunks are taken in bit
// order: of each such pair a pass keeps about one, so that at any time the
// passes of a tile, which start together, are on the same two chunks of G
// and find them in L2 (taken in the order of the ring, the passes were four
// chunks apart and L2 served a third of the requests).
struct AdjChunks {
    uint64_t m0, m1;
    __device__ __forceinline__ static int chunk(int bit, int half) { return (bit >> 1) + (bit & 1) * half; }
    __device__ __forceinline__ int count() const { return __popcll(m0) + __popcll(m1); }
    __device__ __forceinline__ bool has(int bit) const { return (((bit < 64 ? m0 : m1) >> (bit & 63)) & 1) != 0; }
    // the next bit (0 once there is none left; see count())
    __device__ __forceinline__ int pop() {
        if (m0) {
            const int c = __ffsll((unsigned long long)m0) - 1;
            m0 &= m0 - 1;
            return c;
        }
        const int c = m1 ? 63 + __ffsll((unsigned long long)m1) : 0;
        m1 &= m1 - 1;
        return c;
    }
};

// The chunks of NQ emitter blocks from eb0 on: `all` of any of them, `mine` of block
// eb0 + q.
template <int NQ>
__device__ __forceinline__ void adj_chunks(const uint8_t *__restrict__ fl, int nb, int eb0, int q,
                                           AdjChunks &all, AdjChunks &mine) {
    const int lane = threadIdx.x & 63, half = (nb + 1) / 2;
    all = mine = AdjChunks{0, 0};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        if (h && half <= 32) break;   // uniform
        const int bit = 64 * h + lane, c = AdjChunks::chunk(bit, half);
        const bool ok = (bit >> 1) < half && c < nb;
        // (clamped, not guarded, so that the loads are in flight together: BF16,
        // 256 elements / 480^2, three frequencies, 360 -> 343 us, FP32 781 -> 769)
        uint8_t f[NQ];
#pragma unroll
        for (int i = 0; i < NQ; ++i) f[i] = fl[min(eb0 + i, nb - 1) * nb + min(c, nb - 1)];
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const uint64_t b = __ballot(ok && eb0 + i < nb && f[i] != 0);
            (h ? all.m1 : all.m0) |= b;
            if (i == q) (h ? mine.m1 : mine.m0) = b;
        }
    }
}

// The same of eb0 < nb, with the chunks with low-order parts (k_adj_prep) as bits 64
// and up, which rings of up to kAdjLowBlocks blocks do not use otherwise.  A chunk's
// flags are joined before the vote: voted on block by block, with the low-order
// parts, some of the conditions were spilled, and waiting for them took 1 us of each
// workgroup (FP16, four frequencies, 61 elements / 635x317 171 -> 159 us, 272 / 608x304
// 703 -> 655).  In the FP32 kernels this form is the one that spills more (256 / 480^2,
// three frequencies, 720 -> 738 us).
template <int NQ>
__device__ __forceinline__ void adj_chunks_low(const uint8_t *__restrict__ fl, int nb, int eb0, int q,
                                               AdjChunks &all, AdjChunks &mine) {
    const int lane = threadIdx.x & 63, half = (nb + 1) / 2;
    auto flags = [&](int bit, unsigned &a, unsigned &w) {   // of any block, of block eb0 + q
        const int c = AdjChunks::chunk(bit, half);
        const uint8_t *f = fl + min(c, nb - 1);
        a = 0;
#pragma unroll
        for (int i = 0; i < NQ; ++i) a |= f[min(eb0 + i, nb - 1) * nb];   // (row nb - 1 is one of them)
        w = f[min(eb0 + q, nb - 1) * nb];
        const bool ok = (bit >> 1) < half && c < nb;
        a = ok ? a : 0;
        w = ok && eb0 + q < nb ? w : 0;
    };
    unsigned a, w;
    flags(lane, a, w);
    all = AdjChunks{__ballot(a != 0), __ballot(a > 1)};
    mine = AdjChunks{__ballot(w != 0), __ballot(w > 1)};
    if (half > 32) {   // uniform
        flags(64 + lane, a, w);
        all.m1 |= __ballot(a != 0);
        mine.m1 |= __ballot(w != 0);
    }
}

// ------------------------------------------------------------------ FP32, LDS-staged
// Backprojection.  The workgroup owns 64 pixels; its four waves are 2
// (emitter halves) x 2 (pixel halves), each computing 32 e x 32 px of Y per
// chunk of 64 emitters.  Receivers are consumed 32 at a time: the G tile
// [32 r][64 px] (re, im) goes from global memory straight into LDS
// (global_load_lds, 16 bytes per lane), double buffered, so staging costs
// no registers and overlaps the MFMAs of the previous chunk.  Rows are
// unpadded; the 16-byte chunks of row r are XOR-swizzled by (r & 3), which
// puts the four lane groups of a B-fragment read (rows 4 s + kk) on distinct
// banks.  A is stored k-permuted, so a lane's eight A values of a chunk are
// two float4 loads (served from L2: A is shared by every workgroup),
// prefetched one chunk ahead.
constexpr int kAdjNT = 64, kAdjKC = 32, kAdjTile = kAdjKC * 64;
constexpr int kT16NE = 128;   // emitters per pass of the kernels on the 16-bit cores (4 waves x 32)

typedef __attribute__((address_space(3))) void lds_void_t;

// LDS offset (floats) of (tile row r, pixel px) in a swizzled [32][64] tile
__device__ __forceinline__ int adj_off(int r, int px) {
    return r * 64 + ((((px >> 2) ^ ((r & 3) << 2))) << 2) + (px & 3);
}

// Aligned full tiles: wave w fills rows 8 w .. 8 w + 7 of both arrays, four
// rows per instruction.  Lane l of an instruction writes LDS chunk
// (row l / 16, chunk l % 16), so it loads the global chunk that the swizzle
// puts there.  Rows at or beyond m read row m - 1: their A entries are zero.
__device__ __forceinline__ void adj_stage_async(const float *__restrict__ gr, const float *__restrict__ gi, int m,
                                                int64_t N, int rc, int64_t x0, float *sT) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int r0 = wave * 8 + j * 4;
        const int rl = r0 + (lane >> 4);
        const int r = min(rc + rl, m - 1);
        const int gc = (lane & 15) ^ ((rl & 3) << 2);
        const int64_t go = (int64_t)r * N + x0 + 4 * gc;
        __builtin_amdgcn_global_load_lds(gr + go, (lds_void_t *)(sT + r0 * 64), 16, 0, 0);
        __builtin_amdgcn_global_load_lds(gi + go, (lds_void_t *)(sT + kAdjTile + r0 * 64), 16, 0, 0);
    }
}

// Ragged or unaligned tiles: through registers, zero beyond m and N.
__device__ __forceinline__ void adj_stage_regs(const float *__restrict__ gr, const float *__restrict__ gi, int m,
                                               int64_t N, int rc, int64_t x0, float *sT) {
    const int t = threadIdx.x;
    const int rl = t >> 3, r = rc + rl, p0 = (t & 7) * 8;
    float vr[8], vi[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int64_t x = x0 + p0 + q;
        const bool ok = r < m && x < N;
        vr[q] = ok ? gr[(int64_t)r * N + x] : 0.0f;
        vi[q] = ok ? gi[(int64_t)r * N + x] : 0.0f;
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        sT[adj_off(rl, p0 + q)] = vr[q];
        sT[kAdjTile + adj_off(rl, p0 + q)] = vi[q];
    }
}

// NB row blocks starting at b0.  The complex product Y = A conj(G) uses
// three real products, P1 = Ar Gr, P2 = Ai Gi, P3 = (Ar + Ai)(Gr - Gi)
// (Ar + Ai formed in registers), so Yr = P1 + P2 and Yi = P3 - P1 + P2; with
// the Hessian term Z = W |G|^2 (HESS) that is four MFMAs per block and step,
// each on a different accumulator.  Without GRAD, Z alone.
template <int NB, bool GRAD, bool HESS>
__device__ __forceinline__ void adj_mma_steps(const f4 (&va)[2][2], const f4 (&vi)[2][2], const f4 (&vw)[2][2],
                                              const float *sBr, const float *sBi, int kk, const int (&coff)[2],
                                              f4 (&p1)[2][2], f4 (&p2)[2][2], f4 (&p3)[2][2], f4 (&z)[2][2],
                                              int b0) {
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        // B fragments for four steps at a time (one LDS wait per half chunk)
        float br[4][2], bi[4][2];
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
                const int o = (4 * (4 * half + q4) + kk) * 64 + coff[cb];
                br[q4][cb] = sBr[o];
                bi[q4][cb] = sBi[o];
            }
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
        const int s8 = 4 * half + q4;
        float b2[2], bd[2];
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
            if (HESS) b2[cb] = __builtin_fmaf(bi[q4][cb], bi[q4][cb], br[q4][cb] * br[q4][cb]);
            bd[cb] = br[q4][cb] - bi[q4][cb];
        }
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            const int b = b0 + q;
            const float a_r = GRAD ? va[b][s8 >> 2][s8 & 3] : 0.0f, a_i = GRAD ? vi[b][s8 >> 2][s8 & 3] : 0.0f;
            const float a_s = a_r + a_i;
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
                if (GRAD) {
                    p1[b][cb] = MM<float>::mma(a_r, br[q4][cb], p1[b][cb]);
                    p2[b][cb] = MM<float>::mma(a_i, bi[q4][cb], p2[b][cb]);
                    p3[b][cb] = MM<float>::mma(a_s, bd[cb], p3[b][cb]);
                }
                if (HESS) z[b][cb] = MM<float>::mma(vw[b][s8 >> 2][s8 & 3], b2[cb], z[b][cb]);
            }
        }
    }
    }
}

// Where a workgroup's work lies: pixel tile loc.tile(), frequency loc.k().
// A launch over one problem reads them from the grid (blockIdx), a grouped
// launch from the problem table.
struct GridLoc {
    __device__ __forceinline__ int64_t tile() const { return blockIdx.x; }
    __device__ __forceinline__ int k() const { return blockIdx.y; }
    __device__ __forceinline__ int group() const { return 0; }
};
struct ItemLoc {
    int64_t t;
    int kf, q;
    __device__ __forceinline__ int64_t tile() const { return t; }
    __device__ __forceinline__ int k() const { return kf; }
    __device__ __forceinline__ int group() const { return q; }   // emitter-pass group
};

// Kernel argument of a launch over one problem: grid (pixel tiles, frequencies).
struct AdjOne {
    using Loc = GridLoc;
    static constexpr bool kSplit = false;   // one workgroup per (pixel tile, frequency)
    AdjItem item;
    __device__ __forceinline__ const AdjItem &locate(Loc &) const { return item; }
};

// Kernel argument of a launch over one problem whose emitter passes are
// split into item.npg groups: grid (pixel tiles x groups, frequencies), the
// groups of a tile adjacent in logical order and, through the XCD remap, on
// one XCD at about the same time, so that they share its G tiles in L2.
struct AdjOneSplit {
    using Loc = ItemLoc;
    static constexpr bool kSplit = true;
    AdjItem item;
    __device__ __forceinline__ const AdjItem &locate(Loc &loc) const {
        const int64_t l = xcd_remap(blockIdx.x, gridDim.x);
        loc.t = l / item.npg;
        loc.q = (int)(l - loc.t * item.npg);
        loc.kf = blockIdx.y;
        return item;
    }
};

// Kernel argument of a launch over several problems: which problem a flat
// workgroup id belongs to, and its (frequency, pixel tile, group) there.
// Workgroup-uniform.
struct AdjGroupArg {
    using Loc = ItemLoc;
    static constexpr bool kSplit = true;
    AdjGroup G;
    __device__ __forceinline__ const AdjItem &locate(Loc &loc) const {
        const int b = blockIdx.x;
        int j = 0;
        while (j + 1 < G.n && b >= G.item[j + 1].begin) ++j;
        const AdjItem &it = G.item[j];
        const int local = b - it.begin;
        const int per = it.ntiles * it.npg;
        loc.kf = local / per;
        const int rem = local - loc.kf * per;
        loc.t = rem / it.npg;
        loc.q = rem - (int)loc.t * it.npg;
        return it;
    }
};

// HESS = false computes the gradient only (three MFMAs per block and step);
// its registers allow three workgroups per CU (34 KB of LDS each).  The
// argument is one problem (AdjOne: grid = pixel tiles x frequencies) or a
// group of problems (AdjGroup: flat grid over every problem's work items).
// Pixel tile `tile` of frequency k: the partial of emitter-pass group qg of
// npg, its passes [pass0, pass1) of 64 emitters.
// (GRAD without HESS, both, or HESS alone, whose partials go to pg)
template <bool GRAD, bool HESS>
__device__ __forceinline__ void adj_f32_tile(const AdjItem &it, int64_t tile, int k, int npg, int qg, int pass0,
                                             int pass1) {
    const AdjParams &P = it.P;
    const float *__restrict__ Gr = (const float *)it.Gr;
    const float *__restrict__ Gi = (const float *)it.Gi;
    const float *__restrict__ Ar = (const float *)it.Ar;
    const float *__restrict__ Ai = (const float *)it.Ai;
    const float *__restrict__ Wt = (const float *)it.Wt;
    const uint8_t *__restrict__ flags = it.flags;
    double *__restrict__ pg = it.pg;
    double *__restrict__ ph = it.ph;
    __shared__ __align__(16) float sB[2][2 * kAdjTile];   // [buffer][re tile, im tile]
    __shared__ double sred[2][2][kAdjNT];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
    const int row = lane & 15, kk = lane >> 4;
    const int we = wave >> 1, wp = wave & 1;
    const int64_t N = P.N;
    const int64_t x0 = tile * kAdjNT;
    const bool vec = ((N & 3) == 0) && (x0 + kAdjNT <= N);   // workgroup-uniform
    // this lane's column offsets in the swizzled tile (rows 4 s + kk)
    int coff[2];
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) coff[cb] = adj_off(kk, 32 * wp + 16 * cb + row) - kk * 64;
    const int half = (P.nb + 1) / 2;   // see AdjChunks
    double gacc[2] = {0.0, 0.0}, hacc[2] = {0.0, 0.0};

    {
        const float *gr = Gr + (int64_t)k * P.m * N;
        const float *gi = Gi + (int64_t)k * P.m * N;
        const float *ar = Ar + (int64_t)k * P.mp * P.mp;
        const float *ai = Ai + (int64_t)k * P.mp * P.mp;
        const float *wt = Wt + (int64_t)k * P.mp * P.mp;
        const uint8_t *fl = flags + (int64_t)k * P.nb * P.nb;
        // (the diagonal's terms are all of one sign: summed in FP32 per lane they
        // made up most of its error, 3.8e-8 at 100 elements / 92^2, 2.2e-8 so)
        float gp[2] = {0.0f, 0.0f};
        double hp[2] = {0.0, 0.0};
        for (int ec = 64 * pass0; ec < 64 * pass1; ec += 64) {
            f4 p1[2][2], p2[2][2], p3[2][2], z[2][2];
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int c = 0; c < 2; ++c) p1[b][c] = p2[b][c] = p3[b][c] = z[b][c] = f4{0, 0, 0, 0};
            // Chunks of 32 receivers to work on, as wave-uniform bit masks
            // taken before the chunk loop: a flag load inside it would make
            // the MFMAs of a chunk wait for the next chunk's tile, which is
            // issued first.  `all`: of either emitter half (staged), `mine`:
            // of this wave's half.
            AdjChunks all, mine;
            adj_chunks<2>(fl, P.nb, ec >> 5, we, all, mine);
            const int nstep = all.count();
            // The A fragments of the next chunk are loaded during a chunk,
            // along with its G tile, so the MFMAs of a chunk wait only for LDS.
            auto load_a = [&](int rc, f4 (&va)[2][2], f4 (&vi)[2][2], f4 (&vw)[2][2]) {
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    // rows beyond mp (when mp is not a multiple of 64) read row
                    // mp - 1: finite values whose products the epilogue drops
                    const int64_t off = (int64_t)min(ec + 32 * we + 16 * b + row, P.mp - 1) * P.mp + rc + 8 * kk;
                    if (GRAD) {
                        va[b][0] = *reinterpret_cast<const f4 *>(ar + off);
                        va[b][1] = *reinterpret_cast<const f4 *>(ar + off + 4);
                        vi[b][0] = *reinterpret_cast<const f4 *>(ai + off);
                        vi[b][1] = *reinterpret_cast<const f4 *>(ai + off + 4);
                    }
                    if (HESS) {
                        vw[b][0] = *reinterpret_cast<const f4 *>(wt + off);
                        vw[b][1] = *reinterpret_cast<const f4 *>(wt + off + 4);
                    }
                }
            };
            auto stage = [&](int rc, float *dst) {
                if (vec)
                    adj_stage_async(gr, gi, P.m, N, rc, x0, dst);
                else
                    adj_stage_regs(gr, gi, P.m, N, rc, x0, dst);
            };
            f4 va[2][2], vi[2][2], vw[2][2];
            bool on = false;
            if (nstep > 0) {   // workgroup-uniform
                const int bit = all.pop(), c = AdjChunks::chunk(bit, half);
                stage(c * kAdjKC, sB[0]);
                on = mine.has(bit);
                if (on) load_a(c * kAdjKC, va, vi, vw);
            }
            __builtin_amdgcn_s_waitcnt(0);   // this wave's direct-to-LDS loads have landed
            __syncthreads();
            for (int s = 0; s < nstep; ++s) {
                const int buf = s & 1;
                bool on_n = false;
                f4 na[2][2], ni[2][2], nw[2][2];
                if (s + 1 < nstep) {
                    const int bit = all.pop(), c = AdjChunks::chunk(bit, half);
                    stage(c * kAdjKC, sB[buf ^ 1]);
                    on_n = mine.has(bit);
                    if (on_n) load_a(c * kAdjKC, na, ni, nw);
                }
                if (on) adj_mma_steps<2, GRAD, HESS>(va, vi, vw, sB[buf], sB[buf] + kAdjTile, kk, coff, p1, p2, p3, z, 0);
                __builtin_amdgcn_s_waitcnt(0);   // the next chunk has landed in LDS
                __syncthreads();
                on = on_n;
                if (on) {
#pragma unroll
                    for (int b = 0; b < 2; ++b)
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            va[b][h] = na[b][h];
                            vi[b][h] = ni[b][h];
                            vw[b][h] = nw[b][h];
                        }
                }
            }
            // fused epilogue: Re sum_e conj(G_e) Y_e and sum_e |G_e|^2 Z_e.
            // Emitters at or beyond m read row m - 1 (their Y and Z are zero),
            // pixels at or beyond N the last one (dropped below), so that no
            // load waits on a test; a half beyond mp holds rows of another.
            if (ec + 32 * we < P.mp) {   // wave-uniform
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    float ger[4][2], gei[4][2];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int e = min(ec + 32 * we + 16 * b + MM<float>::out_row(kk, i), P.m - 1);
#pragma unroll
                        for (int cb = 0; cb < 2; ++cb) {
                            const int64_t x = min(x0 + 32 * wp + 16 * cb + row, N - 1);
                            ger[i][cb] = gr[(int64_t)e * N + x];
                            gei[i][cb] = gi[(int64_t)e * N + x];
                        }
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
#pragma unroll
                        for (int cb = 0; cb < 2; ++cb) {
                            const float ge_r = ger[i][cb], ge_i = gei[i][cb];
                            if (GRAD) {
                                const float yr = p1[b][cb][i] + p2[b][cb][i];
                                const float yi = (p3[b][cb][i] - p1[b][cb][i]) + p2[b][cb][i];
                                gp[cb] += ge_r * yr + ge_i * yi;
                            }
                            if (HESS) hp[cb] += (double)__builtin_fmaf(ge_i, ge_i, ge_r * ge_r) * (double)z[b][cb][i];
                        }
                    }
                }
            }
        }
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
            gacc[cb] += (double)gp[cb] * P.cg[k];
            hacc[cb] += hp[cb] * P.ch[k];
        }
    }
    // lanes of a column (four groups), then the two emitter halves, in a fixed order
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
        double g = gacc[cb], h = hacc[cb];
        g += __shfl_xor(g, 16);
        h += __shfl_xor(h, 16);
        g += __shfl_xor(g, 32);
        h += __shfl_xor(h, 32);
        if (kk == 0) {
            sred[we][0][32 * wp + 16 * cb + row] = g;
            sred[we][1][32 * wp + 16 * cb + row] = h;
        }
    }
    __syncthreads();
    if (tid < kAdjNT) {
        const int64_t x = x0 + tid;
        if (x < N) {
            const double h = sred[0][1][tid] + sred[1][1][tid];
            pg[((int64_t)k * npg + qg) * N + x] = GRAD ? sred[0][0][tid] + sred[1][0][tid] : h;
            if (GRAD && HESS) ph[((int64_t)k * npg + qg) * N + x] = h;
        }
    }
}

template <bool HESS, typename A, bool GRAD = true>
__global__ void __launch_bounds__(256, GRAD ? (HESS ? 2 : 3) : 4) k_adjoint_f32(const A args) {
    typename A::Loc loc;
    const AdjItem &it = args.locate(loc);
    // one frequency per workgroup (finer work units), and this workgroup's
    // emitter passes (64 emitters each): group qg of npg
    const int npg = A::kSplit ? it.npg : 1, qg = A::kSplit ? loc.group() : 0;
    const int npass = (it.P.mp + 63) / 64;
    adj_f32_tile<GRAD, HESS>(it, loc.tile(), loc.k(), npg, qg, qg * npass / npg, (qg + 1) * npass / npg);
}

// The work items that k_adjoint_split listed, again from the FP32 tables and
// operands: one of its items is two of this kernel's tiles, and each of its
// passes two of this kernel's.
__global__ void __launch_bounds__(256, 3) k_adjoint_f32_list(const AdjItem it) {
    const int n = 2 * it.redo[0];
    const int np16 = (it.P.mp + kT16NE - 1) / kT16NE, np = (it.P.mp + 63) / 64;
    for (int i = blockIdx.x; i < n; i += gridDim.x) {
        const int id = it.redo[1 + (i >> 1)], per = it.ntiles * it.npg;
        const int k = id / per, rem = id - k * per, q = rem % it.npg;
        const int64_t tile = 2 * (int64_t)(rem / it.npg) + (i & 1);
        if (tile * kAdjNT < it.P.N)
            adj_f32_tile<true, false>(it, tile, k, it.npg, q, 2 * (q * np16 / it.npg), min(2 * ((q + 1) * np16 / it.npg), np));
        __syncthreads();   // the next item reuses the LDS
    }
}


// ------------------------------------------------------------------ 16-bit
// |G|^2 of a fragment, rounded to the storage type (products of 16-bit values
// are exact in FP32, so the fused form rounds as a a + b b does; FP16 takes its
// operands without conversions)
template <typename S, typename V>
__device__ __forceinline__ V a16_abs2(V br, V bi) {
    V o;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float a = (float)br[i], b = (float)bi[i];
        o[i] = MM16<S>::from_f(__builtin_fmaf(b, b, __builtin_fmaf(a, a, 0.0f)));
    }
    return o;
}

template <int I>
using Idx = std::integral_constant<int, I>;

// ------------------------------------------------------------------------
// 16-bit backprojection with transposing LDS reads.
//
// Workgroup tile: 128 emitters (a pass; 32 per wave) x 128 pixels, the
// receivers streamed in k-steps of 32.  The G tile of a step (32 receiver
// rows x 128 pixels, both arrays, 16 KB) is copied into LDS by 16-byte direct
// global->LDS loads (one instruction fills four rows), two steps ahead, into
// four buffers.  MFMA B fragments need eight consecutive receivers of one
// pixel per lane; ds_read_b64_tr_b16 delivers four of them from a
// pixel-major tile (within each 16-lane group, lane i receives the i-th
// 16-bit element of the 4 x 8-byte rows its group addressed), so two
// transposing reads give a fragment with no register permutes.  The
// 16-byte chunks of each tile row are XOR-swizzled so that the eight rows
// one half-wave reads together lie on distinct banks; the direct loads
// realise the swizzle by choosing which global chunk each lane fetches.
// A fragments (eight receivers of one emitter) come from L2 as 16-byte
// loads, one step ahead.
//
// The passes of a tile are adjacent workgroups on one XCD, so that they share
// the tile's chunks in L2.  The epilogue loads the pass's own emitter rows
// into the freed tile buffers once more and takes G_e from them with the
// same transposing read (four emitters of one pixel per lane).
constexpr int kT16NT = 128;                   // pixels per tile
constexpr int kT16KC = 32;                    // receivers per k-step
constexpr int kT16Row = 2 * kT16NT;           // bytes per tile row
constexpr int kT16Arr = kT16KC * kT16Row;     // bytes of one array of a tile

typedef short t16v4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) t16v4 t16lds_v4;

// chunk position of 16-byte chunk c in tile row r: c XOR 2 g(r), where g
// numbers the rows {0..3, 8..11} (and their shifts by 4 and 16) 0..7
__device__ __forceinline__ int t16_pos(int r, int c) { return c ^ (2 * ((r & 3) | (((r >> 3) & 1) << 2))); }
// byte offset of (tile row r, pixel px) in one array
__device__ __forceinline__ int t16_off(int r, int px) {
    return r * kT16Row + (t16_pos(r, px >> 3) << 4) + ((px & 7) << 1);
}

// Transposing read: lane (group kk, index i) of the wave addresses row
// r0 + (i >> 2), pixels 4 (i & 3) .. + 3 of a 16-pixel column block; it gets
// rows r0 .. r0 + 3 of pixel (i) of the block.
__device__ __forceinline__ t16v4 t16_tr(const unsigned char *p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((t16lds_v4 *)(p));
}

// The four transposing reads of one column block (rows r and r + 4 of both
// arrays: immediate offsets 0, 4 rows, one array, one array + 4 rows), with
// their wait in the same block.  Written as one asm block so that the
// compiler, which cannot tell these reads from the direct loads filling
// other buffers, adds no wait on those loads here; the k-step's own vmcnt
// wait and barrier order the tile with its reads.
__device__ __forceinline__ void t16_tr4(unsigned addr, t16v4 &a, t16v4 &b, t16v4 &c, t16v4 &d) {
    asm volatile(
        "ds_read_b64_tr_b16 %0, %4\n\t"
        "ds_read_b64_tr_b16 %1, %4 offset:1024\n\t"
        "ds_read_b64_tr_b16 %2, %4 offset:8192\n\t"
        "ds_read_b64_tr_b16 %3, %4 offset:9216\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(a), "=&v"(b), "=&v"(c), "=&v"(d)
        : "v"(addr));
}

// The same for four arrays (k_adjoint_split): eight reads, one wait.
__device__ __forceinline__ void t16_tr8(unsigned addr, t16v4 (&r)[8]) {
    asm volatile(
        "ds_read_b64_tr_b16 %0, %8\n\t"
        "ds_read_b64_tr_b16 %1, %8 offset:1024\n\t"
        "ds_read_b64_tr_b16 %2, %8 offset:8192\n\t"
        "ds_read_b64_tr_b16 %3, %8 offset:9216\n\t"
        "ds_read_b64_tr_b16 %4, %8 offset:16384\n\t"
        "ds_read_b64_tr_b16 %5, %8 offset:17408\n\t"
        "ds_read_b64_tr_b16 %6, %8 offset:24576\n\t"
        "ds_read_b64_tr_b16 %7, %8 offset:25600\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7])
        : "v"(addr));
}

template <typename V>
__device__ __forceinline__ V t16_join(t16v4 lo, t16v4 hi) {
    typedef short s8v __attribute__((ext_vector_type(8)));
    const s8v v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(V, v);
}

// Aligned tiles (N a multiple of 8, m a multiple of 32, 32 N elements
// within 32-bit offsets): of the workgroup's NW waves, wave w issues the
// 16 / NW instructions q from 16 w / NW on of the tile's 16 (array q >> 3, rows 4 (q & 7) .. + 3); `goff[j]` is lane l's
// element offset from the step's first row and pixel (`gr`, `gi`: uniform)
// for its j-th instruction, so the loads take a scalar base and a 32-bit
// lane offset.
template <int NW>
__device__ __forceinline__ void t16_stage_async(const unsigned short *__restrict__ gr,
                                                const unsigned short *__restrict__ gi,
                                                const unsigned *goff, unsigned char *sT) {
    constexpr int NQ = 16 / NW;
    const int q = NQ * __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned short *g = (q >> 3) ? gi : gr;
    unsigned char *d = sT + (q >> 3) * kT16Arr + (q & 7) * 4 * kT16Row;
#pragma unroll
    for (int j = 0; j < NQ; ++j)
        __builtin_amdgcn_global_load_lds(g + goff[j], (lds_void_t *)(d + j * 4 * kT16Row), 16, 0, 0);
}

// Where a direct load will not do (rows that are not 16-byte aligned, a chunk
// with fewer than 32 rows) the same tile goes through registers, loaded during
// the MFMAs of the step before: 16 bytes of row r from pixel x on, in one load
// that needs no alignment unless the table's pixels end within the tile (`full`
// is uniform).  With 2-byte loads, waited for when issued, and now, FP16, two
// frequencies: 130 elements / 301x255 178 -> 93 us, with the Hessian diagonal
// (eight waves, see t16_waves) 292 -> 115, 100 / 256^2 89 -> 51 us, 1000 / 301x255
// (one frequency) 968 -> 392.
typedef unsigned short t16us8 __attribute__((ext_vector_type(8)));
typedef t16us8 t16us8_u __attribute__((aligned(2)));
__device__ __forceinline__ t16us8 t16_load(const unsigned short *__restrict__ g, int r, int64_t N, int64_t x,
                                           bool full) {
    const unsigned short *q = g + (int64_t)r * N;
    if (full) return *reinterpret_cast<const t16us8_u *>(q + x);
    t16us8 v;
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = x + u < N ? q[x + u] : (unsigned short)0;
    return v;
}
// Thread t's part of the tile of rows rc .. rc + 31 (NW waves): pieces t, t +
// 64 NW, .. of 512 an array, piece q being the chunk stored at position q % 16
// of row q / 16.
template <int NW>
__device__ __forceinline__ void t16_load_tile(const unsigned short *__restrict__ gr,
                                              const unsigned short *__restrict__ gi, int m, int64_t N, int rc,
                                              int64_t x0, bool full, t16us8 (&v)[16 / NW]) {
    constexpr int NJ = 16 / NW, RS = 4 * NW;   // pieces a thread; rows they are apart
    const int rl = threadIdx.x >> 4;
    const int64_t x = x0 + 8 * ((threadIdx.x & 15) ^ t16_pos(rl, 0));   // (RS is a multiple of 16)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
        v[j] = t16_load(j * RS >> 5 ? gi : gr, min(rc + rl + (j * RS & 31), m - 1), N, x, full);
}
// ... and into LDS, zero for rows at or beyond m
template <int NW>
__device__ __forceinline__ void t16_store_tile(const t16us8 (&v)[16 / NW], int m, int rc, unsigned char *sT) {
    constexpr int NJ = 16 / NW, RS = 4 * NW;
    const int rl = threadIdx.x >> 4;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int r = rl + (j * RS & 31);
        const t16us8 w = rc + r < m ? v[j] : (t16us8)(unsigned short)0;
        *reinterpret_cast<t16us8 *>(sT + (j * RS >> 5) * kT16Arr + r * kT16Row + (threadIdx.x & 15) * 16) = w;
    }
}

// Waves per workgroup: four of 32 emitters x 128 pixels; with the Hessian
// product eight of 32 x 64, whose accumulators (96 registers) leave two waves
// per SIMD where four of 128 pixels left one.  FP16 / BF16, gradient and
// Hessian diagonal: 130 elements / 301x255, two frequencies, 186 -> 152 us,
// 256 / 480^2, three, 764 -> 675, 1024 / 480^2, one, 1.89 -> 1.68 ms; with
// |G|^2 by fused multiply-adds (20 instead of 44 instructions a fragment in
// FP16) and the sum of its roundings taken off at the end 115, 594 and 1.42 ms.
constexpr int t16_waves(bool hess) { return hess ? 8 : 4; }

template <typename S, bool HESS, bool DIRECT, typename A>
__global__ void __launch_bounds__(64 * t16_waves(HESS), 2) k_adjoint16_tr(const A args) {
    typename A::Loc loc;
    const AdjItem &it = args.locate(loc);
    const AdjParams &P = it.P;
    const S *__restrict__ Ar = (const S *)it.Ar;
    const S *__restrict__ Ai = (const S *)it.Ai;
    const S *__restrict__ Wt = (const S *)it.Wt;
    const uint8_t *__restrict__ flags = it.flags;
    const float *__restrict__ gscale = it.gscale;
    const float *__restrict__ ascale = it.ascale;
    double *__restrict__ pg = it.pg;
    double *__restrict__ ph = it.ph;
    using V = typename MM16<S>::vec;
    constexpr int NW = t16_waves(HESS);
    constexpr int EB = 2;          // 16-row emitter blocks per wave
    constexpr int CB = 32 / NW;    // 16-pixel column blocks per wave
    // four tile buffers as separate LDS objects, addressed by compile-time
    // index inside the k-loop: a direct load into one is then known not to
    // write the one being read
    __shared__ __align__(16) unsigned char sG0[2 * kT16Arr];
    __shared__ __align__(16) unsigned char sG1[2 * kT16Arr];
    __shared__ __align__(16) unsigned char sG2[2 * kT16Arr];
    __shared__ __align__(16) unsigned char sG3[2 * kT16Arr];
    __shared__ float sred[2][4][kT16NT];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int eg = wave & 3, cb0 = wave >> 2 ? CB : 0;   // emitter group, first column block
    const int row = lane & 15, kk = lane >> 4;
    const int64_t N = P.N;
    const int k = loc.k();
    // the last tile ends with the table (its first pixels are the previous one's,
    // and not written), so that every load is whole: as the only one with loads of
    // single values it was what a launch of few tiles waited for
    const int64_t xt = (int64_t)loc.tile() * kT16NT, x0 = max(min(xt, N - kT16NT), (int64_t)0);
    const unsigned short *gr = reinterpret_cast<const unsigned short *>((const S *)it.Gr + (int64_t)k * P.m * N);
    const unsigned short *gi = reinterpret_cast<const unsigned short *>((const S *)it.Gi + (int64_t)k * P.m * N);
    const bool full = x0 + kT16NT <= N;   // uniform; but for tables of fewer pixels
    const S *ar = Ar + (int64_t)k * P.mp * P.mp;
    const S *ai = Ai + (int64_t)k * P.mp * P.mp;
    const S *wt = Wt + (int64_t)k * P.mp * P.mp;
    const uint8_t *fl = flags + (int64_t)k * P.nb * P.nb;
    const int half = (P.nb + 1) / 2;   // see AdjChunks
    const int cmask = half <= 32 ? 63 : 127;   // bits beyond: low-order parts
    auto chunk = [&](int bit) { return AdjChunks::chunk(bit & cmask, half); };
    // lane's element offsets of its four direct-load chunks within a step
    // (of the last tile's chunks beyond N, the last: dropped)
    const int lastc = (int)min(N - 8 - x0, (int64_t)kT16NT);
    unsigned goff[16 / NW];
#pragma unroll
    for (int j = 0; j < 16 / NW; ++j) {
        const int rl = 4 * ((16 / NW * wave + j) & 7) + (lane >> 4);
        goff[j] = (unsigned)(rl * N) + (unsigned)min(8 * ((lane & 15) ^ t16_pos(rl, 0)), lastc);
    }
    // transposing-read offset at rows 8 kk + (row >> 2), pixels 4 (row & 3) of
    // column block 0 (block cb: XOR 32 cb)
    const unsigned t0 = t16_off(8 * kk + (row >> 2), 4 * (row & 3));
    float gp[CB], hp[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) gp[cb] = hp[cb] = 0.0f;
    auto buf = [&](auto itag) -> unsigned char * {
        constexpr int I = decltype(itag)::value & 3;
        return I == 0 ? sG0 : (I == 1 ? sG1 : (I == 2 ? sG2 : sG3));
    };

    const int npass = (P.mp + kT16NE - 1) / kT16NE, npg = it.npg, qg = loc.group();
    const int pass0 = qg * npass / npg, pass1 = (qg + 1) * npass / npg;
    for (int ec = pass0 * kT16NE; ec < pass1 * kT16NE; ec += kT16NE) {
        const int e0 = ec + 32 * eg;
        f4 yr[EB][CB], yn[EB][CB], z[EB][CB];
#pragma unroll
        for (int b = 0; b < EB; ++b)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) yr[b][cb] = yn[b][cb] = z[b][cb] = f4{0, 0, 0, 0};
        // fragments of block (e0 / 32, c); emitter blocks beyond mp read the
        // last one (their Y is dropped)
        const int eb = min(e0 >> 5, P.nb - 1);
        auto load_a = [&](int bit, V (&va)[EB], V (&vi)[EB], V (&vw)[EB]) {
            const int c = chunk(bit);
            const bool lo = bit > cmask;
            const int bi = lo ? c : eb, bj = lo ? eb : c;
            const unsigned co = (unsigned)(bi * P.nb + bj) * 1024u;   // uniform
#pragma unroll
            for (int b = 0; b < EB; ++b) {
                va[b] = *reinterpret_cast<const V *>(ar + co + 512 * b + 8 * lane);
                vi[b] = *reinterpret_cast<const V *>(ai + co + 512 * b + 8 * lane);
                if (HESS) vw[b] = *reinterpret_cast<const V *>(wt + co + 512 * b + 8 * lane);   // (0 for low-order parts)
            }
        };
        // the pass's receiver chunks: `all` of its four waves (staged), `mine`
        // of this wave's 32 emitters
        AdjChunks all, mine;
        adj_chunks_low<4>(fl, P.nb, ec >> 5, eg, all, mine);
        const int nstep = all.count();
        // the chunks of the current step and the next two (opaque to the
        // compiler, which would otherwise keep a strength-reduced address per
        // unrolled step live in registers)
        auto next_bit = [&]() {
            int c = all.pop();
            asm volatile("" : "+s"(c));
            return c;
        };
        int b0 = next_bit(), b1 = next_bit(), b2 = next_bit();
        auto stage = [&](int bit, unsigned char *dst) {
            const int c = chunk(bit);
            t16_stage_async<NW>(gr + ((int64_t)c * kT16KC * N + x0), gi + ((int64_t)c * kT16KC * N + x0), goff, dst);
        };
        t16us8 tv[16 / NW];   // without direct loads: the tile of step s + 1
        auto load_t = [&](int bit) { t16_load_tile<NW>(gr, gi, P.m, N, chunk(bit) * kT16KC, x0, full, tv); };
        // One k-step s (chunk bit b0) on the tile in buffer s mod 4: wait for
        // its tile and its A, issue A of b1 and the tile of step s + 2 (b2),
        // then the MFMAs.  Per step a wave issues A(s + 1) (2 EB or
        // 3 EB loads) and then the tile of s + 2 (16 / NW direct loads), so at the
        // wait only the tile of s + 1 may still be in flight.  `mode` says
        // what the step issues when that is known at compile time (3: A and
        // a tile, 2: A only, 1: nothing; 0: decided from s at run time), so
        // that the compiler's own load-counter waits stay exact.
        auto kstep = [&](int s, auto itag, V (&va)[EB], V (&vi)[EB], V (&vw)[EB], V (&na)[EB], V (&ni)[EB],
                         V (&nw)[EB], auto mode) {
            constexpr int I = decltype(itag)::value;
            constexpr int M = decltype(mode)::value;
            const bool has_a = M == 3 || M == 2 || (M == 0 && s + 1 < nstep);
            const bool has_t = M == 3 || (M == 0 && s + 2 < nstep);
            if (!DIRECT) {
                // the tile of s + 1, read two barriers from now at the latest
                if (has_a) t16_store_tile<NW>(tv, P.m, chunk(b1) * kT16KC, buf(Idx<I + 1>()));
            } else if (has_a) {
                __builtin_amdgcn_s_waitcnt(vmcnt_imm(16 / NW));   // tile s + 1
            } else {
                __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
            }
            lds_barrier();
            const bool on = mine.has(b0);
            if (has_a) load_a(b1, na, ni, nw);
            __builtin_amdgcn_sched_barrier(0);
            if (has_t) {
                if (DIRECT)
                    stage(b2, buf(Idx<I + 2>()));
                else
                    load_t(b2);
            }
            __builtin_amdgcn_sched_barrier(0);
            b0 = b1;
            b1 = b2;
            b2 = next_bit();
            if (!on) return;
            const unsigned char *sb = buf(Idx<I>());
            V nva[EB];
#pragma unroll
            for (int b = 0; b < EB; ++b) nva[b] = neg(vi[b]);
            const unsigned sba = (unsigned)(uintptr_t)(const __attribute__((address_space(3))) unsigned char *)sb;
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                t16v4 r0, r1, i0, i1;
                t16_tr4(sba + (t0 ^ (32u * (cb0 + cb))), r0, r1, i0, i1);
                const V br = t16_join<V>(r0, r1);
                const V bi = t16_join<V>(i0, i1);
                V b2;
                if (HESS) b2 = a16_abs2<S, V>(br, bi);
#pragma unroll
                for (int b = 0; b < EB; ++b) {
                    yr[b][cb] = MM16<S>::mma(va[b], br, yr[b][cb]);
                    yr[b][cb] = MM16<S>::mma(vi[b], bi, yr[b][cb]);
                    yn[b][cb] = MM16<S>::mma(va[b], bi, yn[b][cb]);
                    yn[b][cb] = MM16<S>::mma(nva[b], br, yn[b][cb]);
                    if (HESS) z[b][cb] = MM16<S>::mma(vw[b], b2, z[b][cb]);
                }
            }
        };
        // the k-loop, unrolled by four (buffer index period 4, A registers period 2); the steady state
        // has no conditional steps, the last two to five follow.  (Making
        // those compile-time as well spills the accumulators.)
        auto kloop = [&]() {
            using M3 = std::integral_constant<int, 3>;
            using M2 = std::integral_constant<int, 2>;
            using M1 = std::integral_constant<int, 1>;
            using M0 = std::integral_constant<int, 0>;
            V va[EB], vi[EB], vw[EB], na[EB], ni[EB], nw[EB];
            lds_barrier();   // the previous pass is done with the tile buffers
            if (DIRECT) {
                stage(b0, sG0);
            } else {
                load_t(b0);
                t16_store_tile<NW>(tv, P.m, chunk(b0) * kT16KC, sG0);
            }
            load_a(b0, va, vi, vw);
            // unconditional (a one-chunk pass stages chunk 0, unused), so that
            // the loop is always entered with the same loads in flight and
            // the compiler's load-counter waits at its head stay exact
            if (DIRECT)
                stage(b1, sG1);
            else
                load_t(b1);
            int s = 0;
            for (; s + 6 <= nstep; s += 4) {
                kstep(s, Idx<0>(), va, vi, vw, na, ni, nw, M3());
                kstep(s + 1, Idx<1>(), na, ni, nw, va, vi, vw, M3());
                kstep(s + 2, Idx<2>(), va, vi, vw, na, ni, nw, M3());
                kstep(s + 3, Idx<3>(), na, ni, nw, va, vi, vw, M3());
            }
            if (s < nstep) kstep(s, Idx<0>(), va, vi, vw, na, ni, nw, M0());
            if (s + 1 < nstep) kstep(s + 1, Idx<1>(), na, ni, nw, va, vi, vw, M0());
            if (s + 2 < nstep) kstep(s + 2, Idx<2>(), va, vi, vw, na, ni, nw, M0());
            if (s + 3 < nstep) kstep(s + 3, Idx<3>(), na, ni, nw, va, vi, vw, M0());
            if (s + 4 < nstep) kstep(s + 4, Idx<0>(), va, vi, vw, na, ni, nw, M0());
            // keep the epilogue's work out of the last k-steps' schedule
            __builtin_amdgcn_sched_barrier(0);
        };
        if (nstep > 0) kloop();   // workgroup-uniform
        // fused epilogue: Re sum_e conj(G_e) Y_e and sum_e |G_e|^2 Z_e.  The
        // tile buffers are free once every wave is done with the k-loop:
        // group g's waves copy the chunk of its 32 emitter rows (both arrays)
        // into buffer g again, and a transposing read at rows 16 b + 4 kk gives
        // lane (kk, row) emitters 16 b + 4 kk + i (i = 0..3) of pixel
        // 16 cb + row, the layout of the accumulators (zero beyond m and N).
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
        lds_barrier();
        unsigned char *se = eg == 0 ? sG0 : (eg == 1 ? sG1 : (eg == 2 ? sG2 : sG3));
        const int q1 = NW == 8 ? 8 * (wave >> 2) : 0;   // first of this wave's 64 / NW copies
        if (DIRECT) {
            if (e0 < P.mp) {
                const unsigned short *g0 = gr + ((int64_t)e0 * N + x0), *g1 = gi + ((int64_t)e0 * N + x0);
#pragma unroll
                for (int qq = 0; qq < 64 / NW; ++qq) {
                    const int q = q1 + qq;
                    const int rl = 4 * (q & 7) + (lane >> 4);
                    const unsigned go =
                        (unsigned)(rl * N) + (unsigned)min(8 * ((lane & 15) ^ t16_pos(rl, 0)), lastc);
                    __builtin_amdgcn_global_load_lds((q >> 3) ? g1 + go : g0 + go,
                                                     (lds_void_t *)(se + (q >> 3) * kT16Arr + 4 * (q & 7) * kT16Row),
                                                     16, 0, 0);
                }
            }
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
        } else if (e0 < P.mp) {
            // (rows at or beyond m: the last one, dropped below)
#pragma unroll
            for (int q0 = q1; q0 < q1 + 64 / NW; q0 += 8) {
                t16us8 v[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const int rl = 4 * q + (lane >> 4);
                    v[q] = t16_load(q0 ? gi : gr, min(e0 + rl, P.m - 1), N,
                                    x0 + 8 * ((lane & 15) ^ t16_pos(rl, 0)), full);
                }
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    *reinterpret_cast<t16us8 *>(se + (q0 ? kT16Arr : 0) + 4 * q * kT16Row + 16 * lane) = v[q];
            }
        }
        lds_barrier();
        if (e0 < P.mp) {
#pragma unroll
            for (int b = 0; b < EB; ++b) {
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) {
                    const int off = t16_off(16 * b + 4 * kk + (row >> 2), 16 * (cb0 + cb) + 4 * (row & 3));
                    const t16v4 vr = t16_tr(se + off), vi = t16_tr(se + kT16Arr + off);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const bool ok = e0 + 16 * b + 4 * kk + i < P.m;
                        const float ger = ok ? MM16<S>::bits_to_f((unsigned short)vr[i]) : 0.0f;
                        const float gei = ok ? MM16<S>::bits_to_f((unsigned short)vi[i]) : 0.0f;
                        gp[cb] += ger * yr[b][cb][i] - gei * yn[b][cb][i];
                        if (HESS) {
                            // |G_e|^2 less the rounding error that it has as an operand of
                            // Z: of a pair contracted once one element's |G|^2 is rounded
                            // and counts twice; over the ring each element is about as
                            // often the one as the other, and the errors cancel.  Error
                            // against FP64 with both orders of a pair / with |G_e|^2 / so,
                            // FP16, general weights: 130 elements / 301x255 2.05e-5 / 2.2e-5
                            // / 1.4e-5, 256 / 128^2 1.39e-5 / 1.5e-5 / 0.9e-5, 512 / 96^2 9.4e-6 /
                            // 9.9e-6 / 5.7e-6; BF16 256 / 128^2 1.14e-4 / - / 0.73e-4.
                            const float p = ger * ger + gei * gei;
                            hp[cb] += (2.0f * p - (float)MM16<S>::from_f(p)) * z[b][cb][i];
                        }
                    }
                }
            }
        }
    }
    // the four lane groups of a column, then the emitter groups, in a fixed order
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
        float g = gp[cb], h = hp[cb];
        g += __shfl_xor(g, 16);
        h += __shfl_xor(h, 16);
        g += __shfl_xor(g, 32);
        h += __shfl_xor(h, 32);
        if (kk == 0) {
            sred[0][eg][16 * (cb0 + cb) + row] = g;
            sred[1][eg][16 * (cb0 + cb) + row] = h;
        }
    }
    __syncthreads();
    if (tid < kT16NT) {
        const int64_t x = x0 + tid;
        if (x >= xt && x < N) {
            const double gs = (double)gscale[k], as = ascale[k] > 0.0f ? (double)ascale[k] : 1.0;
            const double g2 = gs * gs;
            double g = 0.0, h = 0.0;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                g += (double)sred[0][w][tid];
                h += (double)sred[1][w][tid];
            }
            const int npgl = it.npg;
            pg[((int64_t)k * npgl + qg) * N + x] = g * (P.cg[k] * g2 * as);
            if (HESS) ph[((int64_t)k * npgl + qg) * N + x] = h * (P.ch[k] * g2 * g2);
        }
    }
}


template <typename A>
void launch_adjoint16(const AdjTask &t, dim3 grid, const A &arg, hipStream_t st) {
    auto go = [&](auto tag, auto hess) {
        using S = decltype(tag);
        constexpr bool H = decltype(hess)::value;
        if (t.direct)
            k_adjoint16_tr<S, H, true><<<grid, 64 * t16_waves(H), 0, st>>>(arg);
        else
            k_adjoint16_tr<S, H, false><<<grid, 64 * t16_waves(H), 0, st>>>(arg);
    };
    if (t.dt == RB_BF16)
        t.hdiag ? go(__hip_bfloat16(), std::true_type()) : go(__hip_bfloat16(), std::false_type());
    else
        t.hdiag ? go(__half(), std::true_type()) : go(__half(), std::false_type());
}

// ------------------------------------------------------------------ FP32 tables on the FP16 matrix cores
// Gradient-only backprojection of FP32 tables with every operand split into
// two FP16 pieces of x s, s a power of two: G s = hi + lo, A s = hi + 2^-12 lo, hi
// the value rounded to FP16, lo the exact remainder (of A, times 2^12) rounded to
// FP16.  hi hi + hi lo + lo (2^-12 hi) on the 16x16x32 FP16 cores (products exact,
// FP32 accumulation) keeps about 22 bits of every product, and an MFMA sums 32
// products at a time instead of 4, so that the result is nearer to FP64 than
// the FP32 cores' (relative L2 error of the gradient, ordered pairs on the FP32 cores
// and so: 256 elements / 480^2, three frequencies, 1.7e-7 -> 1.0e-7, 130 / 301x255, two,
// 1.9e-7 -> 1.3e-7; 65 to 1000 elements, 0.6 to 1.0 of it).
//
// 1024 elements / 1100^2, four frequencies: 105.6 ms on the FP32 cores, 44.3
// ms here (12 MFMAs per complex product of blocks: 1.1 PFLOP/s).  The matrix
// cores are busy 0.53 of the time at 2.0 GHz, to which the card's power limits the
// clock (kernels that draw less run at 2.4); a large FP16 product of the library
// reaches 1.23 PFLOP/s.  256 / 480^2, three frequencies: 1.46
// -> 0.75 ms.  On the way there: rows of G loaded half a chunk ahead 55.1 ms,
// passes four chunks apart (AdjChunks) 64.8 ms.
//
// Scales: A by its largest magnitude per frequency, brought to 2^15; G per
// (frequency, pixel) by its largest magnitude over kSplitRows sampled elements,
// brought to 2^10 (k_adj_colscale).  The pieces hold FP32's bits (a last place of
// 2^-22 or less) of every A s from 2^-14 on and every G s from 2^-2 on, up to
// 65504; the scale of A's low piece is shared out so because residuals range
// further than a pixel's G (1024 elements / 1100^2 phantom: 2^-19 of the largest
// for A, 2^-7 to 2^4.4 of the sample for G).  Whatever lies outside of these
// ranges, but zeros, is computed from FP32 by k_adjoint_f32_list: of a frequency
// with a smaller A all work items, without delay (bad); otherwise those whose
// workgroup has staged such a G.  (Phantom tables have them: in 28 of 1,800 tiles
// at 256 elements, in 172 of 9,454 at 1024, pixels just outside the ring that a few
// elements cover and none of the sampled ones: 1.0 ms for these tiles beside 41.9.)
//
// Workgroup tile, receiver chunks, transposing reads and LDS swizzle are
// those of k_adjoint16_tr; here a chunk's 32 x 128 FP32 tile passes through
// registers (four float4 per array and thread, loaded during the MFMAs of the
// previous chunk), is split there once for all four waves and stored as four
// FP16 arrays of 8 KB, double buffered.
constexpr int kSplitRows = 16, kSplitRowsMore = 128;
typedef _Float16 h4 __attribute__((ext_vector_type(4)));

// scale[k][x] = split_scale(max over the sampled rows of |re|, |im|).  Pixels
// that none of the kSplitRows rows covers (outside the ring, or at its edge,
// where rays end) take kSplitRowsMore rows; 2^100 where those are zero too.
// Also clears what the following launches accumulate into: amax [nf], bad [nf]
// and the list's length.
__global__ void __launch_bounds__(256) k_adj_colscale(int m, int nf, int64_t N, const float *__restrict__ Gr,
                                                      const float *__restrict__ Gi, float *__restrict__ scale,
                                                      float *__restrict__ amax, int *__restrict__ bad,
                                                      int *__restrict__ redo) {
    const int k = blockIdx.y;
    const int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (blockIdx.x == 0 && k == 0) {
        if (threadIdx.x < nf) {
            amax[threadIdx.x] = 0.0f;
            bad[threadIdx.x] = 0;
        }
        if (threadIdx.x == 0) redo[0] = 0;
    }
    if (x >= N) return;
    const float *gr = Gr + (int64_t)k * m * N + x, *gi = Gi + (int64_t)k * m * N + x;
    float top = 0.0f;
#pragma unroll
    for (int q = 0; q < kSplitRows; ++q) {
        const int64_t r = (int64_t)q * m / kSplitRows;
        top = fmaxf(top, fmaxf(fabsf(gr[r * N]), fabsf(gi[r * N])));
    }
    if (!(top > 0.0f)) {
        const int nr = min(m, kSplitRowsMore);
#pragma unroll 8
        for (int q = 0; q < nr; ++q) {
            const int64_t r = (int64_t)q * m / nr;
            top = fmaxf(top, fmaxf(fabsf(gr[r * N]), fabsf(gi[r * N])));
        }
    }
    scale[(int64_t)k * N + x] = top > 0.0f ? split_scale(top, kSplitTopG) : 0x1p100f;
}

template <typename A>
__global__ void __launch_bounds__(256, 2) k_adjoint_split(const A args) {
    typename A::Loc loc;
    const AdjItem &it = args.locate(loc);
    const AdjParams &P = it.P;
    const uint8_t *__restrict__ flags = it.flags;
    double *__restrict__ pg = it.pg;
    constexpr int EB = 2;   // 16-row emitter blocks per wave
    __shared__ __align__(16) unsigned char sT[2][4 * kT16Arr];   // re hi, im hi, re lo, im lo
    __shared__ float sred[4][kT16NT];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row = lane & 15, kk = lane >> 4;
    const int64_t N = P.N;
    const int k = loc.k();
    // (the last tile ends with the table: see k_adjoint16_tr; N is at least a tile)
    const int64_t xt = (int64_t)loc.tile() * kT16NT, x0 = min(xt, N - kT16NT);
    const float *__restrict__ gr = (const float *)it.Gr + (int64_t)k * P.m * N;
    const float *__restrict__ gi = (const float *)it.Gi + (int64_t)k * P.m * N;
    typedef f4 f4_a4 __attribute__((aligned(4)));   // rows need no alignment
    const int64_t per = (int64_t)P.mp * P.mp;
    const _Float16 *__restrict__ ahi = (const _Float16 *)it.split_hi + 2 * k * per;
    const _Float16 *__restrict__ alo = (const _Float16 *)it.split_lo + 2 * k * per;
    const uint8_t *fl = flags + (int64_t)k * P.nb * P.nb;
    const float *__restrict__ sc = it.pscale + (int64_t)k * N;
    const int half = (P.nb + 1) / 2;   // see AdjChunks
    auto list = [&]() {
        it.redo[1 + atomicAdd(it.redo, 1)] = (int)(((int64_t)k * it.ntiles + loc.tile()) * it.npg + loc.group());
    };
    if (it.bad[k]) {   // workgroup-uniform
        if (tid == 0) list();
        return;
    }

    // staging: this thread's four pixels (p4 ..) of tile rows r8 + 8 j
    const int p4 = (tid & 31) * 4, r8 = tid >> 5;
    f4 ps;
#pragma unroll
    for (int q = 0; q < 4; ++q) ps[q] = sc[x0 + p4 + q];
    // of the values this thread has staged (largest of re and im): the largest,
    // and the bits of the smallest but zero, minus one
    float top = 0.0f;
    unsigned low = 0xffffffffu;
    // byte offsets are taken from the chunk's first row and pixel, uniform
    // bases, and fit 32 bits (32 N < 2^30 elements)
    auto at = [](const float *base, unsigned off) {
        return reinterpret_cast<const float *>(reinterpret_cast<const char *>(base) + off);
    };
    const unsigned nb4 = 4u * (unsigned)N;
    auto load = [&](const float *__restrict__ g, int c, f4 (&v)[4]) {
        const float *base = g + (int64_t)c * kT16KC * N + x0;
        const int rl = P.m - 1 - c * kT16KC;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            // rows at or beyond m read row m - 1: their A entries are zero
            const unsigned ro = (unsigned)min(r8 + 8 * j, rl) * nb4;
            v[j] = *reinterpret_cast<const f4_a4 *>(at(base, ro + 4u * p4));
        }
    };
    auto store = [&](const f4 (&vr)[4], const f4 (&vi)[4], unsigned char *d) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int o = t16_off(r8 + 8 * j, p4);
            f4 w[2];
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                const f4 v = a ? vi[j] : vr[j];
                w[a] = v * ps;
                const h4 h = __builtin_convertvector(w[a], h4);
                f4 rem;
#pragma unroll
                for (int q = 0; q < 4; ++q) rem[q] = __builtin_fmaf(v[q], ps[q], -(float)h[q]);
                const h4 l = __builtin_convertvector(rem, h4);
                *reinterpret_cast<h4 *>(d + a * kT16Arr + o) = h;
                *reinterpret_cast<h4 *>(d + (2 + a) * kT16Arr + o) = l;
            }
#pragma unroll
            for (int q = 0; q < 4; q += 2) {
                const float m0 = fmaxf(fabsf(w[0][q]), fabsf(w[1][q])), m1 = fmaxf(fabsf(w[0][q + 1]), fabsf(w[1][q + 1]));
                top = fmaxf(top, fmaxf(m0, m1));
                low = min(low, min(__float_as_uint(m0) - 1u, __float_as_uint(m1) - 1u));
            }
        }
    };
    // transposing-read offset of column block 0, rows 8 kk + (row >> 2);
    // block cb is at t0 ^ 32 cb (the swizzle is an XOR of the chunk number), the
    // rows 4 further on at + 4 kT16Row
    const int t0 = t16_off(8 * kk + (row >> 2), 4 * (row & 3));
    float gp[8];
#pragma unroll
    for (int cb = 0; cb < 8; ++cb) gp[cb] = 0.0f;

    const int npass = (P.mp + kT16NE - 1) / kT16NE, npg = it.npg, qg = loc.group();
    const int pass0 = qg * npass / npg, pass1 = (qg + 1) * npass / npg;
    for (int ec = pass0 * kT16NE; ec < pass1 * kT16NE; ec += kT16NE) {
        const int e0 = ec + 32 * wave;
        f4 yr[EB][8], yn[EB][8];
#pragma unroll
        for (int b = 0; b < EB; ++b)
#pragma unroll
            for (int cb = 0; cb < 8; ++cb) yr[b][cb] = yn[b][cb] = f4{0, 0, 0, 0};
        AdjChunks all, mine;
        adj_chunks<4>(fl, P.nb, ec >> 5, wave, all, mine);
        const int nstep = all.count();
        // fragments [re hi, im hi, re lo, im lo][b] of block (e0 / 32, c)
        const int eblk = min(e0 >> 5, P.nb - 1) * P.nb;
        auto load_a = [&](int c, h8 (&a)[4][EB]) {
            const int64_t o = (int64_t)(eblk + c) * 2048 + 8 * lane;
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int b = 0; b < EB; ++b)
                    a[t][b] = *reinterpret_cast<const h8 *>((t < 2 ? ahi : alo) + o + 1024 * (t & 1) + 512 * b);
        };
        auto mma_cb = [&](unsigned sba, const h8 (&a)[4][EB], const h8 (&n)[2][EB], int cb) {
            using M = MM16<__half>;
            t16v4 r[8];
            t16_tr8(sba + (unsigned)(t0 ^ (32 * cb)), r);
            h8 b0 = t16_join<h8>(r[0], r[1]), b1 = t16_join<h8>(r[2], r[3]);
            const h8 b2 = t16_join<h8>(r[4], r[5]), b3 = t16_join<h8>(r[6], r[7]);
            auto term = [&](const h8 (&x)[EB], const h8 &u, const h8 (&y)[EB], const h8 &v) {
#pragma unroll
                for (int b = 0; b < EB; ++b) {
                    yr[b][cb] = M::mma(x[b], u, yr[b][cb]);
                    yn[b][cb] = M::mma(y[b], v, yn[b][cb]);
                }
            };
            term(a[0], b0, a[0], b1);
            term(a[1], b1, n[0], b0);
            term(a[0], b2, a[0], b3);
            term(a[1], b3, n[0], b2);
            b0 *= (_Float16)(1.0f / kSplitLoA);   // exact from 2^-2 on
            b1 *= (_Float16)(1.0f / kSplitLoA);
            term(a[2], b0, a[2], b1);
            term(a[3], b1, n[1], b0);
        };
        // the MFMAs of the chunk in buffer s mod 2
        auto mma = [&](int s, const h8 (&a)[4][EB]) {
            const unsigned sba =
                (unsigned)(uintptr_t)(const __attribute__((address_space(3))) unsigned char *)sT[s & 1];
            h8 n[2][EB];
#pragma unroll
            for (int b = 0; b < EB; ++b) {
                n[0][b] = neg(a[1][b]);
                n[1][b] = neg(a[3][b]);
            }
#pragma unroll
            for (int cb = 0; cb < 8; ++cb) mma_cb(sba, a, n, cb);
        };
        // The steps but the last issue the next chunk's loads without a
        // condition, so that the compiler's load-counter waits stay exact: the
        // rows of G at the start, used at the end, and A, whose registers are
        // in use until then, before the conversions.
        auto kloop = [&]() {
            f4 vr[4], vi[4];
            h8 a[4][EB];
            int bit = all.pop(), c = AdjChunks::chunk(bit, half);
            load(gr, c, vr);
            load(gi, c, vi);
            load_a(c, a);
            lds_barrier();   // the previous pass is done with the tile buffers
            store(vr, vi, sT[0]);
            int s = 0;
            for (; s + 1 < nstep; ++s) {
                lds_barrier();   // chunk s is in LDS, and no wave still reads the other buffer
                const bool on = mine.has(bit);
                bit = all.pop();
                c = AdjChunks::chunk(bit, half);
                load(gr, c, vr);
                load(gi, c, vi);
                __builtin_amdgcn_sched_barrier(0);
                if (on) mma(s, a);
                load_a(c, a);
                __builtin_amdgcn_sched_barrier(0);
                store(vr, vi, sT[(s & 1) ^ 1]);
            }
            lds_barrier();
            if (mine.has(bit)) mma(s, a);
        };
        if (nstep > 0) kloop();   // workgroup-uniform
        // fused epilogue: Re sum_e conj(G_e) Y_e, with G_e in FP32.  Rows at or
        // beyond m read row m - 1 (their Y is zero).
        if (e0 < P.mp) {   // wave-uniform
            const float *br = gr + (int64_t)e0 * N + x0, *bi = gi + (int64_t)e0 * N + x0;
            const int rl = P.m - 1 - e0;
#pragma unroll
            for (int b = 0; b < EB; ++b) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const unsigned ro = (unsigned)min(16 * b + 4 * kk + i, rl) * nb4;
                    float ger[8], gei[8];
#pragma unroll
                    for (int cb = 0; cb < 8; ++cb) {
                        const unsigned o = ro + 4u * (unsigned)(16 * cb + row);
                        ger[cb] = *at(br, o);
                        gei[cb] = *at(bi, o);
                    }
#pragma unroll
                    for (int cb = 0; cb < 8; ++cb) gp[cb] += ger[cb] * yr[b][cb][i] - gei[cb] * yn[b][cb][i];
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
    }
    // (a scale below 2^-60: G_e Y could leave FP32's range before it is taken back)
    const float smin = fminf(fminf(ps[0], ps[1]), fminf(ps[2], ps[3]));
    const int beyond = __syncthreads_or(!(top < kSplitMax) || low < __float_as_uint(kSplitMinG) - 1u || smin < 0x1p-60f);
    if (beyond && tid == 0) list();
    // the four lane groups of a column, then the waves, in a fixed order
#pragma unroll
    for (int cb = 0; cb < 8; ++cb) {
        float g = gp[cb];
        g += __shfl_xor(g, 16);
        g += __shfl_xor(g, 32);
        if (kk == 0) sred[wave][16 * cb + row] = g;
    }
    __syncthreads();
    if (tid < kT16NT) {
        const int64_t x = x0 + tid;
        if (x >= xt) {
            const double g = ((double)sred[0][tid] + (double)sred[1][tid]) +
                             ((double)sred[2][tid] + (double)sred[3][tid]);
            const double s = (double)split_scale(it.ascale[k], kSplitTopA) * (double)sc[x];
            pg[((int64_t)k * npg + qg) * N + x] = g * P.cg[k] / s;
        }
    }
}

// grad += sum_k sum_q pg[k][q], hd += sum_k sum_q ph[k][q] in frequency
// order, then emitter-pass group order.
__global__ void k_adj_sum(int64_t N, int nf, int npg, const double *__restrict__ pg, const double *__restrict__ ph,
                          double *__restrict__ grad, double *__restrict__ hd) {
    const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= N) return;
    double g = 0.0, h = 0.0;
    for (int k = 0; k < nf * npg; ++k) {
        g += pg[(int64_t)k * N + x];
        if (hd) h += ph[(int64_t)k * N + x];
    }
    grad[x] += g;
    if (hd) hd[x] += h;
}

}  // namespace

// ---------------------------------------------------------------- host side
// rows/columns of the adjoint operands are padded to a multiple of 32
constexpr int kRedoBlocks = 768;   // of k_adjoint_f32_list: three per compute unit

static int pad_m(int m) { return (m + 31) / 32 * 32; }

static AdjParams adj_params(const rb_geometry *g, const double *freqs, int nf) {
    AdjParams P;
    P.m = g->m;
    P.mp = pad_m(g->m);
    P.nb = P.mp / 32;
    P.N = (int64_t)g->nx * g->ny;
    P.nf = nf;
    const double dA = g->h * g->h;
    for (int k = 0; k < nf; ++k) {
        const double om = 2.0 * M_PI * freqs[k];
        const double c = om * om * dA;
        P.cg[k] = 2.0 * c;       // 2: the operands hold half of A + A^T and W + W^T
        P.ch[k] = 2.0 * c * c;
    }
    return P;
}

struct AdjWs {
    void *Ar, *Ai, *Wt;
    uint8_t *flags;
    float *ascale;
    double *pg, *ph;  // per-frequency partials of the f32 backprojection
};

// Workgroups that split the emitter passes of one pixel tile: every pass
// (64 emitters in the FP32 kernel, 128 in the 16-bit one) goes to a
// workgroup of its own once there are four or more, the passes of a tile
// adjacent in logical order and on one XCD (AdjOneSplit), so that the
// tile's G rows come from HBM once and from L2 for the other passes (measured
// while every ordered pair was contracted, FP32 cores, 1024 elements / 1100^2: 221.6 ->
// 209.6 ms per 4-frequency launch; 16-bit: 51.9 -> 47.6 ms).  Ordering the split workgroups pass-major instead (all
// workgroups in flight on one pass, sharing its W.D rows) was slower: 224.7
// and 60.0 ms; so was nothing in between: dealing a tile's groups into 2
// or 4 subsets on their own XCDs (each L2 then holds a half or a quarter of
// W.D) left the launches at 211.8 / 212.3 ms (FP32, from 211.5) and 33.2 /
// 33.4 ms (16-bit, from 33.5).  One workgroup per tile otherwise.
static int adj_groups(const rb_geometry *g, rb_dtype dt) {
    if (dt == RB_F32) {
        const int npass = (pad_m(g->m) + 63) / 64;   // 64 emitters per pass of k_adjoint_f32
        return npass >= 4 ? npass : 1;
    }
    if (dt != RB_BF16 && dt != RB_F16) return 1;
    const int ne = kT16NE;   // emitters per pass of k_adjoint16_tr
    const int npass = (pad_m(g->m) + ne - 1) / ne;
    return npass >= 4 ? npass : 1;
}

// Length of an AdjItem's bad and redo together.
static size_t split_ints(const rb_geometry *g, int nf, rb_dtype dt) {
    return RB_MAX_NF + 1 + (size_t)nf * blocks_for((int64_t)g->nx * g->ny, kT16NT) * adj_groups(g, dt);
}

// Whether a gradient-only FP32 problem takes k_adjoint_split: from 65
// elements (a pass has 128, and at 64 half of its waves are idle) and with
// more workgroups than compute units.  us per call, k_adjoint_f32 against
// k_adjoint_split, two frequencies: 64 elements / 480^2 129 / 134, 80 / 480^2
// 254 / 168, 96 / 128^2 (256 workgroups) 27 / 31, 96 / 256^2 82 / 61, 128 /
// 256^2 106 / 73, 130 / 301x255 238 / 117, 256 / 181^2 187 / 89, 512 / 480^2 2873 /
// 1363; one frequency, 256 / 128x150 (300 workgroups) 54 / 50.
static bool adj_split(const rb_geometry *g, int nf, rb_dtype dt) {
    if (dt != RB_F32 || g->m <= 64) return false;
    const int npass = (pad_m(g->m) + kT16NE - 1) / kT16NE;
    const int64_t tiles = blocks_for((int64_t)g->nx * g->ny, kT16NT);
    if (nf * tiles * (adj_groups(g, dt) > 1 ? npass : 1) <= 256) return false;
    // 32-bit offsets within 32 rows; a whole tile
    if ((int64_t)g->nx * g->ny >= (int64_t)1 << 25 || (int64_t)g->nx * g->ny < kT16NT) return false;
    // its high operands live in place of W, the low ones and the scales in
    // the Hessian partials, neither of which a gradient needs
    const int64_t mp = pad_m(g->m), N = (int64_t)g->nx * g->ny;
    Carver c(nullptr, 0);
    c.take<_Float16>((size_t)nf * 2 * mp * mp);
    c.take<float>((size_t)nf * N);
    c.take<int>(split_ints(g, nf, dt));
    return c.used <= (size_t)nf * adj_groups(g, dt) * N * sizeof(double);
}

static AdjWs carve_adj(Carver &c, const rb_geometry *g, int nf, rb_dtype dt) {
    const int mp = pad_m(g->m);
    const size_t npg = (size_t)adj_groups(g, dt);
    const size_t per = (size_t)nf * mp * mp;
    const size_t es = dt == RB_F64 ? 8 : (dt == RB_F32 ? 4 : 2);
    AdjWs w;
    w.Ar = c.take<char>(per * es);
    w.Ai = c.take<char>(per * es);
    w.Wt = c.take<char>(per * es);
    w.flags = c.take<uint8_t>((size_t)nf * (mp / 32) * (mp / 32));
    w.ascale = c.take<float>(RB_MAX_NF);
    w.pg = c.take<double>((size_t)nf * npg * g->nx * g->ny);
    w.ph = c.take<double>((size_t)nf * npg * g->nx * g->ny);
    return w;
}

size_t adjoint_workspace_bytes(const rb_geometry *g, int nf, rb_dtype dt) {
    Carver c(nullptr, 0);
    carve_adj(c, g, nf, dt);
    return c.used + 256;
}

rb_status adjoint_prepare(const rb_geometry *g, const void *G_re, const void *G_im, const float *gscale,
                          rb_dtype dt, const double *freqs, int nf, const double *d_res, const double *w_data,
                          double *grad, double *hdiag, void *ws, size_t ws_bytes, hipStream_t st, AdjTask *task) {
    if (ws_bytes < adjoint_workspace_bytes(g, nf, dt)) {
        set_error("adjoint workspace too small: need %zu bytes", adjoint_workspace_bytes(g, nf, dt));
        return RB_ENOMEM;
    }
    Carver c(ws, ws_bytes);
    AdjWs w = carve_adj(c, g, nf, dt);
    AdjParams P = adj_params(g, freqs, nf);
    const dim3 gp(P.nb * P.nb, nf);
    AdjItem &it = task->item;
    it.P = P;
    it.Gr = G_re;
    it.Gi = G_im;
    it.Ar = w.Ar;
    it.Ai = w.Ai;
    it.Wt = w.Wt;
    it.flags = w.flags;
    it.gscale = gscale;
    it.ascale = w.ascale;
    it.pg = w.pg;
    it.ph = w.ph;
    it.begin = 0;
    it.split_hi = it.split_lo = nullptr;
    it.pscale = nullptr;
    it.redo = it.bad = nullptr;
    if (hdiag && adj_split(g, nf, dt)) {
        // The Hessian diagonal by itself, its one product on the FP32 cores,
        // before the gradient's pieces take the place of W (gradient and
        // diagonal as four products there, and so: 1024 elements / 1100^2, four
        // frequencies, 156 -> 89 ms, 256 / 480^2, three, 2.18 -> 1.44, 96 / 256^2,
        // two, 113 -> 105 us)
        k_adj_prep<float, false, 1><<<gp, 256, 0, st>>>(g->m, P.mp, d_res, w_data, nullptr, (float *)w.Ar,
                                                        (float *)w.Ai, (float *)w.Wt, w.flags);
        RB_LAUNCHED();
        it.npg = adj_groups(g, dt);
        it.ntiles = (int)blocks_for(P.N, kAdjNT);
        if (it.npg == 1)
            k_adjoint_f32<true, AdjOne, false><<<dim3(it.ntiles, nf), 256, 0, st>>>(AdjOne{it});
        else
            k_adjoint_f32<true, AdjOneSplit, false><<<dim3((unsigned)it.ntiles * it.npg, nf), 256, 0, st>>>(
                AdjOneSplit{it});
        RB_LAUNCHED();
        k_adj_sum<<<blocks_for(P.N, 256), 256, 0, st>>>(P.N, nf, it.npg, it.pg, nullptr, hdiag, nullptr);
        RB_LAUNCHED();
        hdiag = nullptr;
    }
    task->split = !hdiag && adj_split(g, nf, dt);
    // (32 N elements within 32-bit offsets)
    task->direct = (dt == RB_BF16 || dt == RB_F16) && P.N % 8 == 0 && P.m % kT16KC == 0 && P.N < ((int64_t)1 << 26);
    if (task->split) {
        Carver h(w.ph, (size_t)-1);
        it.split_hi = w.Wt;
        it.split_lo = h.take<_Float16>((size_t)nf * 2 * P.mp * P.mp);
        float *ps = h.take<float>((size_t)nf * P.N);
        it.pscale = ps;
        it.bad = h.take<int>(split_ints(g, nf, dt));
        it.redo = it.bad + RB_MAX_NF;
        k_adj_colscale<<<dim3(blocks_for(P.N, 256), nf), 256, 0, st>>>(
            g->m, nf, P.N, (const float *)G_re, (const float *)G_im, ps, w.ascale, it.bad, it.redo);
        RB_LAUNCHED();
        k_adj_amax<<<gp, 256, 0, st>>>(g->m, P.nb, d_res, w_data, reinterpret_cast<unsigned *>(w.ascale));
        RB_LAUNCHED();
    }
    if (dt == RB_BF16 || dt == RB_F16) {
        RB_TRY(fill_f32(w.ascale, 0.0f, nf, st));
        k_adj_amax<<<gp, 256, 0, st>>>(g->m, P.nb, d_res, w_data, reinterpret_cast<unsigned *>(w.ascale));
        RB_LAUNCHED();
    }
    switch (dt) {
        case RB_F64:
            k_adj_prep<double, false><<<gp, 256, 0, st>>>(g->m, P.mp, d_res, w_data, nullptr, (double *)w.Ar,
                                                          (double *)w.Ai, (double *)w.Wt, w.flags);
            break;
        case RB_F32:
            k_adj_prep<float, false, 1><<<gp, 256, 0, st>>>(g->m, P.mp, d_res, w_data, w.ascale, (float *)w.Ar,
                                                               (float *)w.Ai, (float *)w.Wt, w.flags,
                                                               (_Float16 *)it.split_hi, (_Float16 *)it.split_lo, it.bad);
            break;
        case RB_BF16:
            k_adj_prep<__hip_bfloat16, true, 2><<<gp, 256, 0, st>>>(g->m, P.mp, d_res, w_data, w.ascale,
                                                                 (__hip_bfloat16 *)w.Ar, (__hip_bfloat16 *)w.Ai,
                                                                 (__hip_bfloat16 *)w.Wt, w.flags);
            break;
        case RB_F16:
            k_adj_prep<__half, true, 2><<<gp, 256, 0, st>>>(g->m, P.mp, d_res, w_data, w.ascale, (__half *)w.Ar,
                                                         (__half *)w.Ai, (__half *)w.Wt, w.flags);
            break;
    }
    RB_LAUNCHED();
    it.ntiles = (int)blocks_for(P.N, dt == RB_F32 && !task->split ? kAdjNT : kT16NT);
    // (fewer than four passes of k_adjoint_f32: one group, as carved)
    it.npg = task->split && adj_groups(g, dt) > 1 ? (P.mp + kT16NE - 1) / kT16NE : adj_groups(g, dt);
    task->dt = dt;
    task->grad = grad;
    task->hdiag = hdiag;
    return RB_OK;
}

rb_status adjoint_run(const AdjTask &task, hipStream_t st) {
    const AdjItem &it = task.item;
    const AdjParams &P = it.P;
    const int nf = P.nf;
    double *grad = task.grad, *hdiag = task.hdiag;
    switch (task.dt) {
        case RB_F64: {
            auto go = [&](auto rb, auto cb, auto hess) {
                k_adjoint<double, decltype(rb)::value, decltype(cb)::value, decltype(hess)::value>
                    <<<dim3(blocks_for(P.N, 64 * decltype(cb)::value), nf), 256, 0, st>>>(
                        P, (const double *)it.Gr, (const double *)it.Gi, (const double *)it.Ar,
                        (const double *)it.Ai, (const double *)it.Wt, it.flags, it.pg, it.ph);
            };
            // 128 pixels a workgroup once those are two per compute unit
            const bool wide = (int64_t)blocks_for(P.N, 128) * nf >= 512;
            if (hdiag)
                wide ? go(Idx<2>(), Idx<2>(), std::true_type()) : go(Idx<2>(), Idx<1>(), std::true_type());
            else
                wide ? go(Idx<2>(), Idx<2>(), std::false_type()) : go(Idx<2>(), Idx<1>(), std::false_type());
            RB_LAUNCHED();
            k_adj_sum<<<blocks_for(P.N, 256), 256, 0, st>>>(P.N, nf, 1, it.pg, it.ph, grad, hdiag);
            break;
        }
        case RB_F32: {
            if (task.split) {
                k_adjoint_split<<<dim3((unsigned)it.ntiles * it.npg, nf), 256, 0, st>>>(AdjOneSplit{it});
                RB_LAUNCHED();
                k_adjoint_f32_list<<<kRedoBlocks, 256, 0, st>>>(it);
            } else if (it.npg == 1) {
                dim3 ga(blocks_for(P.N, kAdjNT), nf);
                const AdjOne one{it};
                if (hdiag)
                    k_adjoint_f32<true><<<ga, 256, 0, st>>>(one);
                else
                    k_adjoint_f32<false><<<ga, 256, 0, st>>>(one);
            } else {
                dim3 ga((unsigned)it.ntiles * it.npg, nf);
                const AdjOneSplit one{it};
                if (hdiag)
                    k_adjoint_f32<true><<<ga, 256, 0, st>>>(one);
                else
                    k_adjoint_f32<false><<<ga, 256, 0, st>>>(one);
            }
            RB_LAUNCHED();
            k_adj_sum<<<blocks_for(P.N, 256), 256, 0, st>>>(P.N, nf, it.npg, it.pg, it.ph, grad, hdiag);
            break;
        }
        case RB_BF16:
        case RB_F16: {
            launch_adjoint16(task, dim3((unsigned)it.ntiles * it.npg, nf), AdjOneSplit{it}, st);
            RB_LAUNCHED();
            k_adj_sum<<<blocks_for(P.N, 256), 256, 0, st>>>(P.N, nf, it.npg, it.pg, it.ph, grad, hdiag);
            break;
        }
    }
    RB_LAUNCHED();
    return RB_OK;
}

rb_status adjoint_run_grouped(AdjTask *const *tasks, int n, hipStream_t st) {
    // contraction type and variant of a task: f32 / bf16 / f16, FP32 on the
    // FP16 cores, 16-bit with direct loads, with or without the Hessian
    // diagonal; f64 runs alone
    auto kind = [](const AdjTask &t) {
        return 8 * (int)t.dt + (t.direct ? 4 : 0) + (t.split ? 2 : 0) + (t.hdiag ? 1 : 0);
    };
    bool done[256] = {};
    RB_CHECK_ARG(n >= 0 && n <= 256, "grouped backprojection: %d problems (at most 256)", n);
    for (int i = 0; i < n; ++i) {
        if (done[i]) continue;
        if (tasks[i]->dt == RB_F64) {
            RB_TRY(adjoint_run(*tasks[i], st));
            done[i] = true;
            continue;
        }
        // up to kAdjGroupMax not-yet-run tasks of this kind, in order
        AdjGroupArg arg;
        AdjGroup &G = arg.G;
        G.n = 0;
        int idx[kAdjGroupMax];
        int64_t blocks = 0;
        for (int j = i; j < n && G.n < kAdjGroupMax; ++j) {
            if (done[j] || kind(*tasks[j]) != kind(*tasks[i])) continue;
            AdjItem it = tasks[j]->item;
            it.begin = (int)blocks;
            blocks += (int64_t)it.ntiles * it.npg * it.P.nf;
            G.item[G.n] = it;
            idx[G.n++] = j;
            done[j] = true;
        }
        RB_CHECK_ARG(blocks < (int64_t)1 << 31, "grouped backprojection: too many workgroups");
        const bool hess = tasks[i]->hdiag != nullptr;
        switch (tasks[i]->dt) {
            case RB_F32:
                if (tasks[i]->split) {
                    k_adjoint_split<<<(unsigned)blocks, 256, 0, st>>>(arg);
                    RB_LAUNCHED();
                    for (int q = 0; q < G.n; ++q) {
                        k_adjoint_f32_list<<<kRedoBlocks, 256, 0, st>>>(tasks[idx[q]]->item);
                        RB_LAUNCHED();
                    }
                } else if (hess)
                    k_adjoint_f32<true><<<(unsigned)blocks, 256, 0, st>>>(arg);
                else
                    k_adjoint_f32<false><<<(unsigned)blocks, 256, 0, st>>>(arg);
                break;
            case RB_BF16:
            case RB_F16:
                launch_adjoint16(*tasks[i], dim3((unsigned)blocks), arg, st);
                break;
            default:
                break;
        }
        RB_LAUNCHED();
        for (int q = 0; q < G.n; ++q) {
            const AdjTask &t = *tasks[idx[q]];
            k_adj_sum<<<blocks_for(t.item.P.N, 256), 256, 0, st>>>(t.item.P.N, t.item.P.nf, t.item.npg, t.item.pg,
                                                                   t.item.ph, t.grad, t.hdiag);
            RB_LAUNCHED();
        }
    }
    return RB_OK;
}

rb_status adjoint_impl(const rb_geometry *g, const void *G_re, const void *G_im, const float *gscale,
                       rb_dtype dt, const double *freqs, int nf, const double *d_res, const double *w_data,
                       double *grad, double *hdiag, void *ws, size_t ws_bytes, hipStream_t st) {
    AdjTask task;
    RB_TRY(adjoint_prepare(g, G_re, G_im, gscale, dt, freqs, nf, d_res, w_data, grad, hdiag, ws, ws_bytes, st,
                           &task));
    return adjoint_run(task, st);
}

// ---------------------------------------------------------------- no-allocation variant
// Scratch of rb_born_adjoint_weighted_noalloc: the same workspace the
// ordinary entry point carves from its caller's buffer, held in one device
// array per GPU (allocated when the library is loaded on that GPU and kept
// until the process ends).  Host code never passes `scratch` itself to a
// kernel: its name there is a host-side stand-in; the device address comes
// from hipGetSymbolAddress, looked up once per device.
static __device__ __align__(256) unsigned char scratch[RB_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};
}  // namespace

// Device address of `scratch` on the current device.
static rb_status scratch_address(void **out) {
    int dev = 0;
    RB_HIP(hipGetDevice(&dev));
    RB_CHECK_ARG(dev >= 0 && dev < kMaxDevices, "device index %d out of range", dev);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        RB_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return RB_OK;
}

}  // namespace rb

extern "C" {

size_t rb_adjoint_workspace_bytes(const rb_geometry *g, int32_t nf, rb_dtype dtype) {
    if (rb::check_geometry(g) != RB_OK || nf < 1 || nf > RB_MAX_NF) return 0;
    return rb::adjoint_workspace_bytes(g, nf, dtype);
}

rb_status rb_born_adjoint_weighted(const rb_geometry *g, const void *G_re, const void *G_im, const float *scale,
                                   rb_dtype dtype, const double *freqs_hz, int32_t nf, const double *d_res,
                                   const double *w_data, double *grad, double *hdiag, void *ws, size_t ws_bytes,
                                   void *stream) {
    rb::clear_error();
    RB_TRY(rb::check_contraction(g, G_re, G_im, scale, dtype, freqs_hz, nf));
    RB_CHECK_ARG(d_res && w_data && grad, "d_res/w_data/grad are NULL");
    RB_CHECK_ARG(ws, "workspace is NULL");
    return rb::adjoint_impl(g, G_re, G_im, scale, dtype, freqs_hz, nf, d_res, w_data, grad, hdiag, ws, ws_bytes,
                            rb::as_stream(stream));
}

rb_status rb_born_adjoint_weighted_noalloc(const rb_geometry *g, const void *G_re, const void *G_im,
                                           const float *scale, rb_dtype dtype, const double *freqs_hz,
                                           int32_t nf, const double *d_res, const double *w_data, double *grad,
                                           double *hdiag, void *stream) {
    rb::clear_error();
    RB_TRY(rb::check_contraction(g, G_re, G_im, scale, dtype, freqs_hz, nf));
    RB_CHECK_ARG(d_res && w_data && grad, "d_res/w_data/grad are NULL");
    const size_t need = rb::adjoint_workspace_bytes(g, nf, dtype);
    if (need > (size_t)RB_NOALLOC_SCRATCH_BYTES) {
        rb::set_error("rb_born_adjoint_weighted_noalloc: this problem needs %zu bytes of scratch, the fixed "
                      "scratch holds %zu (use rb_born_adjoint_weighted with a workspace)",
                      need, (size_t)RB_NOALLOC_SCRATCH_BYTES);
        return RB_ENOMEM;
    }
    void *ws = nullptr;
    RB_TRY(rb::scratch_address(&ws));
    return rb::adjoint_impl(g, G_re, G_im, scale, dtype, freqs_hz, nf, d_res, w_data, grad, hdiag, ws,
                            (size_t)RB_NOALLOC_SCRATCH_BYTES, rb::as_stream(stream));
}

}  // extern "C"
