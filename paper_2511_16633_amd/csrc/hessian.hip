// Diagonal of the Gauss-Newton Hessian (paper, Inverse Problem section,
// Eq. 10; the single-step paragraph's weights) for data weights of the form
// the inversion uses: receiver selection by circular distance (Results:
// the opposite part of the ring) with some selected pairs zeroed (Results:
// the largest values of a frequency set set to zero),
//     W_er = [d(e, r) >= dmin] - [(e, r) zeroed],
//     hd(x) = sum_k omega_k^4 h^4 sum_e g_e(x) sum_r W_er g_r(x),  g = |G|^2.
// With S = sum_r g_r and B_e = sum_{d(e,r) < dmin} g_r (the band the
// selection removes), sum_r W_er g_r = S - B_e - sum_{r zeroed for e} g_r,
// so a pixel costs O(m + zeroed pairs) instead of the O(m^2) of a dense W:
// B_e is a circular window sum that slides by one receiver per emitter.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "born.h"
#include "common.h"

namespace rb {
namespace {

template <typename T>
__device__ __forceinline__ double to_d(T v) { return (double)v; }
template <>
__device__ __forceinline__ double to_d<__hip_bfloat16>(__hip_bfloat16 v) { return (double)__bfloat162float(v); }
template <>
__device__ __forceinline__ double to_d<__half>(__half v) { return (double)__half2float(v); }

constexpr int kHbThreads = 256;
template <int I>
using Int = std::integral_constant<int, I>;

// four 16-bit table values loaded together (a row may start at any pixel)
typedef unsigned hb_u2 __attribute__((ext_vector_type(2)));
typedef hb_u2 hb_u2_u __attribute__((aligned(2)));
template <typename T>
__device__ __forceinline__ float quad_value(hb_u2 q, int i) {
    const unsigned short b = (unsigned short)(q[i >> 1] >> (16 * (i & 1)));
    return (float)to_d(__builtin_bit_cast(T, b));
}

struct HbParams {
    int m, nf, dmin, zcap;
    int64_t N;
    double ch[RB_MAX_NF];   // omega^4 h^4
};

// A block holds PB pixels; its NT threads form NG = NT / PB groups per pixel.
// g for the block's pixels is staged in LDS as [r][PB] values of type L,
// and every sum is taken in L: FP64 for FP64 tables, else FP32 (the
// precision of the matrix-core path).  Group q owns the receivers and emitters
// [q per, (q + 1) per), per = ceil(m / NG); the sums of the groups'
// receivers make up S and the whole groups of a group's first window; partial
// sums are combined in group order, so the result is deterministic.
// (Whole rows of a group, not one in NG, are what lets a first window be put
// together from 6 group sums and 38 rows in place of 255 at 1024 elements.)
//
// With AHEAD (RM at least per) a frequency's rows are loaded into registers during
// the sums of the one before: one block of 1024 threads fills a compute unit, which otherwise
// reads memory for a third of the time only (1024 elements, four
// frequencies, 1 % zeroed: FP32 / 1100^2 18.1 -> 14.2 ms, BF16 / 480^2 3.35 ->
// 2.46).  The zeroed pairs pass through
// LDS in chunks of 2 NT, double-buffered, packed as e << 16 | r (0xffffffff
// for an entry out of range), one barrier per chunk; the first ZN chunks
// are loaded ahead of the next frequency's rows, so that waiting for them does
// not wait for the rows.  With FP32 sums
// and PB a multiple of 4 (ZQ) a thread takes four pixels of a zeroed pair
// at once (one 16-byte LDS read per element instead of four 4-byte ones):
// the pairs are then packed as row offsets (e PQ) << 16 | r PQ in units of
// four pixels, an entry out of range pointing at a row of zeros after the
// m rows of g, and the partial sums of the 4 NG pair groups are combined
// per pixel in group order through the chunk buffer.  Workgroups go to the
// XCDs in contiguous pixel ranges, so the table rows of neighbouring
// workgroups (64 or 128 bytes each) share L2 lines.
template <typename T, typename L, int PB, int RM, bool AHEAD, int NT = kHbThreads>
__global__ void __launch_bounds__(NT, AHEAD ? 4 : 1) k_hess_band(HbParams P, const T *__restrict__ Gr,
                                                  const T *__restrict__ Gi, const float *__restrict__ gscale,
                                                  const int2 *__restrict__ zeroed,
                                                  const int *__restrict__ nzero, double *__restrict__ hd) {
    constexpr int NG = NT / PB;
    constexpr bool ZQ = PB % 4 == 0 && sizeof(L) == 4;
    constexpr int PQ = ZQ ? PB / 4 : 1;       // pixel quads per row
    extern __shared__ __align__(16) unsigned char lds_raw[];
    L *sg = reinterpret_cast<L *>(lds_raw);   // [m][PB], with ZQ one more row of zeros
    __shared__ L spart[NT];
    constexpr int ZC = 2 * NT;                // zeroed pairs per chunk
    constexpr int ZN = NT / kHbThreads;       // chunks loaded ahead
    __shared__ __align__(16) unsigned sz[2][ZC];   // two chunks of the zeroed-pair list, packed
    const int m = P.m;
    const int t = threadIdx.x;
    const int px = t % PB, grp = t / PB;
    const int64_t xb = xcd_remap(blockIdx.x, gridDim.x) * PB;   // the block's first pixel
    if (ZQ && t < PB) sg[m * PB + t] = 0;     // ordered before its readers by the barriers below
    const int64_t x = xb + px;
    const bool okx = x < P.N;
    const int64_t xc = min(x, P.N - 1);       // pixels beyond N: the last one, dropped
    // 16-bit tables load whole pixel quads (block-uniform; with
    // 2-byte loads the load phase was bound by instruction issue: 1024
    // elements / 1100^2 bf16, 17.8 -> 12.6 ms per 4-frequency launch, while
    // FP32 tables gained nothing and keep one pixel per thread)
    constexpr bool VQ = ZQ && sizeof(T) == 2;
    const bool quads = VQ && xb + PB <= P.N;
    const L *col = sg + px;
    const int half = P.dmin - 1;              // band: r = e + s, |s| <= half
    const bool none = 2 * half + 1 >= m;      // the band covers the ring: nothing selected
    const int per = (m + NG - 1) / NG, nseg = (m + per - 1) / per;
    const int e0 = per * grp, e1 = min(m, e0 + per);   // (empty for the last groups)
    auto seg_len = [&](int q) { return min(per, m - q * per); };
    double total = 0.0;

    // the rows of one frequency: RM rows of this pixel, or (quads) RM / 4 rows
    // of four pixels, RGN apart; rows at or beyond m read the last one
    constexpr int RGN = NT / PQ, RQ = VQ ? RM / 4 : 1, RS = VQ || !AHEAD ? 1 : RM;
    const int pq = t % PQ, rg = t / PQ;
    hb_u2 qa[RQ], qb[RQ];
    T va[RS], vb[RS];
    auto load = [&](int k) {
        const T *gr = Gr + (int64_t)k * m * P.N, *gi = Gi + (int64_t)k * m * P.N;
        // (opaque: else RM addresses would be kept from frequency to frequency)
        int r0 = VQ ? rg : e0;
        asm volatile("" : "+v"(r0));
        if constexpr (VQ) {
            if (!quads) return;
#pragma unroll
            for (int u = 0; u < RQ; ++u) {
                const int64_t o = (int64_t)min(r0 + u * RGN, m - 1) * P.N + xb + 4 * pq;
                qa[u] = *reinterpret_cast<const hb_u2_u *>(gr + o);
                qb[u] = *reinterpret_cast<const hb_u2_u *>(gi + o);
            }
        } else {
            int64_t o = (int64_t)min(r0, m - 1) * P.N + xc;
#pragma unroll
            for (int u = 0; u < RS; ++u) {
                va[u] = gr[o];
                vb[u] = gi[o];
                o += r0 + u + 1 < m ? P.N : 0;
            }
        }
    };
    auto mag2 = [](L a, L b, L sc) { return (a * a + b * b) * sc; };
    auto frequency = [&](int k, auto last) {
        const L sc = gscale ? (L)gscale[k] * (L)gscale[k] : (L)1;
        L sp = 0;
        if constexpr (VQ) {
            if (quads) {
#pragma unroll
                for (int u = 0; u < RQ; ++u) {
                    const int r = rg + u * RGN;
                    if (r < m) {
                        float4 v;
                        v.x = mag2(quad_value<T>(qa[u], 0), quad_value<T>(qb[u], 0), sc);
                        v.y = mag2(quad_value<T>(qa[u], 1), quad_value<T>(qb[u], 1), sc);
                        v.z = mag2(quad_value<T>(qa[u], 2), quad_value<T>(qb[u], 2), sc);
                        v.w = mag2(quad_value<T>(qa[u], 3), quad_value<T>(qb[u], 3), sc);
                        *reinterpret_cast<float4 *>(sg + r * PB + 4 * pq) = v;
                    }
                }
            } else {   // the block of the table's last pixels
                const T *gr = Gr + (int64_t)k * m * P.N + xc, *gi = Gi + (int64_t)k * m * P.N + xc;
#pragma unroll 8
                for (int r = e0; r < e1; ++r) 
                    sg[r * PB + px] = mag2((L)to_d(gr[(int64_t)r * P.N]), (L)to_d(gi[(int64_t)r * P.N]), sc);
            }
            lds_barrier();
#pragma unroll 8
            for (int r = e0; r < e1; ++r) sp += col[r * PB];
        } else if constexpr (!AHEAD) {   // RM rows in flight
            const T *gr = Gr + (int64_t)k * m * P.N + xc, *gi = Gi + (int64_t)k * m * P.N + xc;
            for (int r0 = e0; r0 < e1; r0 += RM) {
                T wa[RM], wb[RM];
#pragma unroll
                for (int u = 0; u < RM; ++u) {
                    wa[u] = gr[(int64_t)min(r0 + u, m - 1) * P.N];
                    wb[u] = gi[(int64_t)min(r0 + u, m - 1) * P.N];
                }
#pragma unroll
                for (int u = 0; u < RM; ++u) {
                    if (r0 + u < e1) {
                        const L v = mag2((L)to_d(wa[u]), (L)to_d(wb[u]), sc);
                        sg[(r0 + u) * PB + px] = v;
                        sp += v;
                    }
                }
            }
        } else {
#pragma unroll
            for (int u = 0; u < RS; ++u) {
                if (e0 + u < e1) {
                    const L v = mag2((L)to_d(va[u]), (L)to_d(vb[u]), sc);
                    sg[(e0 + u) * PB + px] = v;
                    sp += v;
                }
            }
        }
        spart[t] = sp;
        lds_barrier();
        // the zeroed pairs of the first chunks, then the next frequency's rows
        const int nz = nzero ? min(nzero[k], P.zcap) : 0;   // block-uniform
        const int2 *zk = zeroed + (int64_t)k * P.zcap;
        // (m PQ < 2^16: PB = 32 only for m <= 1024)
        const unsigned zoff = ((unsigned)(m * PQ) << 16) | (unsigned)(m * PQ);   // the row of zeros
        unsigned zr[ZN][2];
        auto fetch = [&](int c0) {
            int2 q[ZN][2];
#pragma unroll
            for (int c = 0; c < ZN; ++c)
#pragma unroll
                for (int h = 0; h < 2; ++h) q[c][h] = zk[min(c0 + c * ZC + h * NT + t, nz - 1)];
#pragma unroll
            for (int c = 0; c < ZN; ++c)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int2 p = q[c][h];
                    const bool ok = c0 + c * ZC + h * NT + t < nz && (unsigned)p.x < (unsigned)m && (unsigned)p.y < (unsigned)m;
                    zr[c][h] = ZQ ? (ok ? ((unsigned)(p.x * PQ) << 16) | (unsigned)(p.y * PQ) : zoff)
                                  : (ok ? ((unsigned)p.x << 16) | (unsigned)p.y : 0xffffffffu);
                }
        };
        if (nz > 0) fetch(0);
        if (AHEAD && !decltype(last)::value) load(k + 1);
        L S = 0;
#pragma unroll 8
        for (int q = 0; q < NG; ++q) S += spart[q * PB + px];
        L acc = 0;
        if (!none && e0 < e1) {
            // window of e0: receivers e0 - half .. e0 + half (mod m), fewer
            // than m of them; whole groups by their sums
            L B = 0;
            if (half >= 0) {
                int n = half + 1, q = grp;   // e0, e0 + 1, ..
                while (n >= seg_len(q)) {
                    B += spart[q * PB + px];
                    n -= seg_len(q);
                    if (++q == nseg) q = 0;
                }
#pragma unroll 8
                for (int i = 0; i < n; ++i) B += col[(q * per + i) * PB];
                n = half, q = grp ? grp - 1 : nseg - 1;   // e0 - 1, e0 - 2, ..
                while (n >= seg_len(q)) {
                    B += spart[q * PB + px];
                    n -= seg_len(q);
                    q = q ? q - 1 : nseg - 1;
                }
                const int end = q * per + seg_len(q);
#pragma unroll 8
                for (int i = 1; i <= n; ++i) B += col[(end - i) * PB];
            }
            // slide: add e + half + 1, drop e - half
            int ra = e0 + half + 1, rd = e0 - half;
            if (ra >= m) ra -= m;
            if (rd < 0) rd += m;
#pragma unroll 4
            for (int e = e0; e < e1; ++e) {
                acc += col[e * PB] * (S - B);
                if (half >= 0) {
                    B += col[ra * PB] - col[rd * PB];
                    if (++ra == m) ra = 0;
                    if (++rd == m) rd = 0;
                }
            }
        }
        // zeroed pairs.  ZQ: thread (gz, pq) sums pairs gz (mod 4 NG) for
        // pixels 4 pq .. 4 pq + 3
        const int gz = t / PQ;
        const float4 *cq = reinterpret_cast<const float4 *>(sg) + pq;
        float4 zs = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        auto chunk = [&](int c0, const unsigned (&reg)[2], int b) {
            sz[b][t] = reg[0];
            sz[b][NT + t] = reg[1];
            lds_barrier();   // chunk b is in LDS; the chunk read two rounds ago is done
            const int cn = min(ZC, nz - c0);
            if constexpr (ZQ) {
                constexpr int NGZ = NT / PQ, ZU = 2;   // pairs in flight a thread
                for (int i0 = gz; i0 < cn; i0 += ZU * NGZ) {
                    float4 fa[ZU], fb[ZU];
#pragma unroll
                    for (int u = 0; u < ZU; ++u) {
                        const int i = i0 + u * NGZ;
                        const unsigned q = i < cn ? sz[b][i] : zoff;
                        fa[u] = cq[q >> 16];
                        fb[u] = cq[q & 0xffffu];
                    }
#pragma unroll
                    for (int u = 0; u < ZU; ++u) {
                        zs.x += fa[u].x * fb[u].x;
                        zs.y += fa[u].y * fb[u].y;
                        zs.z += fa[u].z * fb[u].z;
                        zs.w += fa[u].w * fb[u].w;
                    }
                }
            } else {
                for (int i0 = grp; i0 < cn; i0 += 8 * NG) {
                    L pr[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int i = i0 + u * NG;
                        pr[u] = 0;
                        if (i < cn) {
                            const unsigned q = sz[b][i];
                            if (q != 0xffffffffu) pr[u] = col[(int)(q >> 16) * PB] * col[(int)(q & 0xffffu) * PB];
                        }
                    }
#pragma unroll
                    for (int u = 0; u < 8; ++u) acc -= pr[u];
                }
            }
        };
        for (int s0 = 0; s0 < nz; s0 += ZN * ZC) {
            if (s0 > 0) fetch(s0);
#pragma unroll
            for (int c = 0; c < ZN; ++c)
                if (s0 + c * ZC < nz) chunk(s0 + c * ZC, zr[c], (ZN == 1 ? s0 / ZC : c) & 1);
        }
        lds_barrier();   // every thread has read spart, sg and sz
        if constexpr (ZQ) {
            // the 4 NG pair groups' partial sums, [gz][PB] in the chunk
            // buffer; pixel px of group grp takes groups 4 grp .. 4 grp + 3
            float *zp = reinterpret_cast<float *>(&sz[0][0]);
            if (nz > 0) {
                reinterpret_cast<float4 *>(zp)[gz * PQ + pq] = zs;
                lds_barrier();
                const float *zc = zp + 4 * grp * PB + px;
                acc -= ((zc[0] + zc[PB]) + zc[2 * PB]) + zc[3 * PB];
            }
        }
        spart[t] = acc;
        lds_barrier();
        if (grp == 0) {
            L a = 0;
#pragma unroll 8
            for (int q = 0; q < NG; ++q) a += spart[q * PB + px];
            total += (double)a * P.ch[k];
        }
        lds_barrier();
    };
    if (AHEAD) load(0);
    for (int k = 0; k + 1 < P.nf; ++k) frequency(k, std::false_type());
    frequency(P.nf - 1, std::true_type());
    if (grp == 0 && okx) hd[x] += total;
}

// LDS of the [m][PB] values (and the row of zeros): within 40 KiB for
// blocks of 256 threads, 140 KiB for the wide blocks (whose static arrays
// take up to 20 KiB more)
constexpr size_t kHbLds = 40960, kHbLdsWide = 143360;
// the wide blocks: pixels and threads
constexpr int kHbWidePB = 32, kHbWideNT = 1024;

}  // namespace

rb_status hessian_band_impl(const rb_geometry *g, const void *G_re, const void *G_im, const float *gscale,
                            rb_dtype dt, const double *freqs, int nf, int dmin, const int *zeroed,
                            const int *nzero, int zcap, double *hdiag, hipStream_t st) {
    HbParams P;
    P.m = g->m;
    P.nf = nf;
    P.N = (int64_t)g->nx * g->ny;
    P.dmin = dmin;
    P.zcap = zcap;
    // pixels per block: [m][pb] values within 40 KiB.  For 256 < m <= 1024
    // and 32/16-bit tables a block of 1024 threads keeps 32 pixels (up to
    // 128 KiB of LDS): reads of a table row then span 64 or 128 bytes
    // instead of 16 or 32.  Rows a thread loads at once: all of its rows up to 16, half
    // of them beyond (rounded up to even; a load beyond a thread's rows is one too
    // many).  us with 8 or 16 by the ring's size alone / all / half / a third, FP32,
    // two frequencies: 100 elements / 256^2 29.4 / 27.3 / 29.4 / 31.2, 130 / 728^2 (one)
    // 156.6 / - / 123.8 / 124.1, 160 / 480^2 159.7 / - / 126.6 / 132.2, 256 / 480^2
    // (three) 310 / - / 310 / 336 (64 pixels a block: 362); FP64 500 / 256^2 8 / 16 rows
    // 278 / 443.  A frequency ahead where one block fills a compute unit and for
    // 16-bit tables, whose rows take half the registers (256 elements, BF16 351
    // -> 229 us; FP32 330 -> 362).
    const bool f64 = dt == RB_F64;
    const bool wide = !f64 && P.m > 256 && P.m <= 1024;
    const int pb = f64 ? (P.m <= 256 ? 16 : (P.m <= 1024 ? 4 : 1)) : (P.m <= 1024 ? kHbWidePB : 2);
    const bool zq = !f64 && pb % 4 == 0;   // the kernel's ZQ: one more row
    const size_t lds = (size_t)(P.m + (zq ? 1 : 0)) * pb * (f64 ? sizeof(double) : sizeof(float));
    if (lds > (wide ? kHbLdsWide : kHbLds)) {
        set_error("m = %d is too large for the banded Hessian", P.m);
        return RB_EUNSUPPORTED;
    }
    const double dA = g->h * g->h;
    for (int k = 0; k < nf; ++k) {
        const double om = 2.0 * M_PI * freqs[k];
        const double c = om * om * dA;
        P.ch[k] = c * c;
    }
    const unsigned nb = (unsigned)((P.N + pb - 1) / pb);
    const int2 *z = reinterpret_cast<const int2 *>(zeroed);
    if (zcap == 0) nzero = nullptr;
    auto go = [&](auto tag, auto ltag, const float *gs) {
        using T = decltype(tag);
        using L = decltype(ltag);
        const T *gr = static_cast<const T *>(G_re), *gi = static_cast<const T *>(G_im);
        auto launch = [&](auto pbt, auto rmt, auto ahead, auto ntt) {
            constexpr int PB = decltype(pbt)::value, RM = decltype(rmt)::value, NT = decltype(ntt)::value;
            auto kfn = k_hess_band<T, L, PB, RM, decltype(ahead)::value, NT>;
            if (NT > kHbThreads)
                (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kfn),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            kfn<<<nb, NT, lds, st>>>(P, gr, gi, gs, z, nzero, hdiag);
        };
        // (rows a thread loads: m over the groups)
        const Int<kHbThreads> nt;
        const std::true_type ahead;
        const std::false_type now;
        // ... at once (see above)
        auto rows = [&](auto pbt, int rm) {
            switch ((rm + 1) / 2 * 2) {
                case 2: case 4: launch(pbt, Int<4>(), now, nt); break;
                case 6: launch(pbt, Int<6>(), now, nt); break;
                case 8: launch(pbt, Int<8>(), now, nt); break;
                case 10: launch(pbt, Int<10>(), now, nt); break;
                case 12: launch(pbt, Int<12>(), now, nt); break;
                case 14: launch(pbt, Int<14>(), now, nt); break;
                default: launch(pbt, Int<16>(), now, nt); break;
            }
        };
        const int per = (P.m + kHbThreads / pb - 1) / (kHbThreads / pb);
        if constexpr (std::is_same<T, double>::value) {
            if (pb == 16)
                rows(Int<16>(), per);
            else if (pb == 4)
                launch(Int<4>(), Int<8>(), now, nt);
            else
                launch(Int<1>(), Int<8>(), now, nt);
        } else if (wide) {
            const Int<kHbWideNT> wnt;
            if (P.m <= 512)
                launch(Int<32>(), Int<16>(), ahead, wnt);
            else if (P.m <= 768)
                launch(Int<32>(), Int<24>(), ahead, wnt);
            else
                launch(Int<32>(), Int<32>(), ahead, wnt);
        } else if (pb == 2) {
            launch(Int<2>(), Int<16>(), now, nt);
        } else if constexpr (sizeof(T) == 4) {
            rows(Int<32>(), per > 16 ? (per + 1) / 2 : per);
        } else if (P.m <= 64) {
            launch(Int<32>(), Int<8>(), ahead, nt);
        } else if (P.m <= 128) {
            launch(Int<32>(), Int<16>(), ahead, nt);
        } else {
            launch(Int<32>(), Int<32>(), ahead, nt);
        }
    };
    switch (dt) {
        case RB_F64: go(double(), double(), nullptr); break;
        case RB_F32: go(float(), float(), nullptr); break;
        case RB_BF16: go(__hip_bfloat16(), float(), gscale); break;
        case RB_F16: go(__half(), float(), gscale); break;
    }
    RB_LAUNCHED();
    return RB_OK;
}

}  // namespace rb

extern "C" {

rb_status rb_born_hessian_banded(const rb_geometry *g, const void *G_re, const void *G_im, const float *scale,
                                 rb_dtype dtype, const double *freqs_hz, int32_t nf, int32_t dmin,
                                 const int32_t *zeroed, const int32_t *nzero, int32_t zcap, double *hdiag,
                                 void *stream) {
    rb::clear_error();
    RB_TRY(rb::check_contraction(g, G_re, G_im, scale, dtype, freqs_hz, nf));
    RB_CHECK_ARG(hdiag != nullptr, "hdiag is NULL");
    RB_CHECK_ARG(dmin >= 0, "dmin must be >= 0");
    RB_CHECK_ARG(zcap >= 0 && (zcap == 0 || (zeroed && nzero)), "zeroed/nzero are required when zcap > 0");
    return rb::hessian_band_impl(g, G_re, G_im, scale, dtype, freqs_hz, nf, dmin, zeroed, nzero, zcap, hdiag,
                                 rb::as_stream(stream));
}

}  // extern "C"
