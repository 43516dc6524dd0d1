// The streaming MPdist-profile kernel: eqs. 9-13 of section 4.1 for every
// (query, window), with nothing of the distance matrix or of its sliding row
// minima in global memory except the few rows that decide a window's value.
//
// A workgroup takes a strip: one query (w rows) against the SBW windows from
// C0, i.e. the w x (SBW + w - 1) block of y = (1 - rho) / 2 in [0, 1] (see
// pst_profile.hip: the same anchors, recurrence and clamp, cell for cell, so
// the results are the same bits).  k-th smallest of a window's 2w values
// (eq. 13) is found in two passes over the block:
//
//   1. Every thread owns V = 6 adjacent columns and walks down the rows; the
//      covariance moves one column right per row (a wave shift).  Column
//      minima (eq. 10) stay in registers; of the rows only the minima of
//      groups of G columns are kept, in LDS.
//   2. For each block of G windows: a row's sliding minimum (eq. 11) at every
//      window of the block lies between the minimum over the groups that
//      cover the block's windows (U) and the minimum over the whole groups
//      inside all of them (C); a column minimum counts from the first window
//      that holds it.  The k-th smallest U and the k-th smallest C bound the
//      block's values: lo <= v <= hi, whatever the data.  Rows and columns
//      with C < lo are below every v, those with U > hi above; the others
//      (about a tenth of the rows) are listed.  In a third to a half of the
//      blocks lo = hi and v is known.
//   3. The rows are walked again and the listed (row, group) pieces of y are
//      kept (global scratch, compact, so that most of it stays in L2).
//   4. Each listed row's sliding minima over its block, one lane per row; then
//      each window's selection among its block's listed values: a sorting
//      network per window where the list is short, counts over the wave where
//      it is long.
//
// Exact for any input: nothing is guessed that is not a bound.
//
// What bounds it: at w <= 178 VALU issue, past it latency (two or four waves a
// SIMD, few enough that no unit is full).  Vector instructions per 64 cells, their
// share of the issue rate and bytes of HBM traffic a cell (k_profile: 42, 0.42 and
// 9.9 at w = 129, and held by the traffic), and ms against k_profile's:
//   w = 33, 50 000 points of a regime series    104   0.70   8.4    4.9 /  6.4
//   w = 129, 100 000                             38   0.75   3.1    6.5 / 12.6
//   w = 257, a walk of 200 000                   35   0.44   7.0   40.6 / 52
//   w = 513, 100 003                             26   0.34   4.0    9.9 / 18.8
//
// A strip's windows reach w-1 columns into the next strip, and the column
// minima there are the next strip's (k_profile's rule, except at the end of a
// tile of 8 strips): a workgroup walks a run of strips right to left and keeps
// those minima; before a run that ends inside a tile it walks the first w-1
// columns of the strip to its right.
#include "pst_internal.h"

#include <algorithm>

// A build with -DPST_PROBE adds up each wave's time between phase marks and a
// few counts (pst_stream_probe_read); for analysis only.
#ifdef PST_PROBE
__device__ unsigned long long g_stream_probe[16 * 64];
#define PROBE_ADD(i, c)                                                                             \
    do {                                                                                            \
        if ((threadIdx.x & 63) == 0)                                                                \
            atomicAdd(&g_stream_probe[(i) * 64 + (blockIdx.x & 63)], (unsigned long long)(c));      \
    } while (0)
#define PROBE_MARK(v) const long long v = clock64()
#define PROBE_SPAN(i, v) PROBE_ADD(i, clock64() - (v))
#else
#define PROBE_ADD(i, c) ((void)0)
#define PROBE_MARK(v) ((void)0)
#define PROBE_SPAN(i, v) ((void)0)
#endif

namespace pst {
namespace {

constexpr int V = 6;                 // columns per thread
constexpr int VA = 7;                // diagonals per thread while anchoring
constexpr int WCOL = 64 * V;         // columns of a wave
constexpr int RCH = 6;               // rows per step of a pass
constexpr int kMaxNT = 448;          // threads of the widest strip
constexpr int kSelect = 64 * 25;     // listed values that a wave holds in LDS
constexpr int kSelectPad = 32 * 49;  // read past them, never used
constexpr int kKeep = 32;            // keys of a long list that a lane keeps
constexpr int kOpen = 64;            // open items of a block with one upper half that are looked at whole
constexpr int kMaxRank = 16;         // smallest keys that a lane keeps of a block
constexpr uint32_t kOne = 0x3F800000u;   // key of y = 1, the largest
constexpr uint32_t kNone = 0xFFFFFFFFu;  // never counted

// Columns per group: at most w/2, so that every window holds a whole group, and
// small against w, so that a block's bounds stay tight, while the group minima
// of a strip leave LDS for the next workgroup.  For w =
// 179 .. 264 (strips of 1984 windows, two workgroups a CU; of 992 beside jobs past
// w = 513) they are kept as
// their upper 16 bits, rounded down: 24 columns in the space of 48 (w = 257,
// 100 000 points, l = 256: 11.2 -> 9.3 ms; 200 000 points of a walk: 61 -> 46).
// Wider strips fill a CU's LDS either way; there whole keys of 48 columns are
// faster (w = 513: 10.7 against 12.0 ms, half the blocks to bound).
__host__ __device__ inline int stream_group(int w) {
    return w < 24 ? 6 : (w < 80 ? 12 : (w <= 264 ? 24 : 48));
}
__host__ __device__ inline bool stream_half(int w) { return w > kStreamNarrow && w <= 264; }
constexpr int kHalfShift = 14;       // keys are at most kOne = 0x3F800000

struct StreamArgs {
    ProfileBatch B;     // tile_end counts runs
    int32_t SBW;
    int32_t run;        // strips of a run, a divisor of `tile`
    int32_t tile;       // strips of a tile
    int32_t tail;       // the last job's queries from here are taken strip by strip
};
static_assert(sizeof(StreamArgs) <= 4000, "kernel arguments must fit the 4 KB limit");

// Sizes of a strip of w rows in a workgroup of NT threads.
struct Dims {
    int NW, NC, NG, NGW, ldg, nblk, items, cap;
    __host__ __device__ Dims(int G, bool half, int w, int NT, int SBW) {
        NW = NT / 64;
        NC = NT * V;                       // columns of the workgroup's threads
        NG = (SBW + w - 1 + G - 1) / G;    // groups with columns of the strip
        NGW = (NG + 15) / 16;              // words of a row's groups to keep
        // row stride of the group minima, one past the end; odd in words (lanes = rows)
        ldg = half ? 2 * (((NG + 2) / 2) | 1) : (NG + 1) | 1;
        nblk = (SBW + G - 1) / G;          // blocks of G windows
        items = 2 * w + G - 1;             // rows and columns of a block's windows
        cap = 64 * (half ? 9 : (G == 48 ? 18 : (G + 3) / 4));   // listed values a wave holds in scratch
    }
};

// LDS of a strip, in floats.
struct Lds {
    int rst, bnd, col, carry, need, blk, bm, total, wp;
    __host__ __device__ Lds(bool half, int w, const Dims &d) {
        wp = (w + RCH + 3) & ~3;
        rst = 0;                                 // float4 [w]: {inv/2, df, dg, h/2}
        bnd = rst + 4 * w;                       // [NW][wp] covariance left of each wave's columns
        col = bnd + d.NW * wp;                   // [NC] anchors of row 0, then column minima
        carry = col + d.NC;                      // [2][w] column minima of the strip to the right
        need = carry + 2 * w;                    // [w][NGW] 16 groups to keep, slots before them << 16
        blk = need + w * d.NGW;                  // [nblk] {lo, hi, below, listed}
        blk = (blk + 3) & ~3;
        bm = blk + 4 * d.nblk;                   // [w][ldg] group minima; the anchors' staging before
        const int lists = d.NW * kSelect + kSelectPad;   // later each wave's listed values
        const int mins = ((half ? w * d.ldg / 2 : w * d.ldg) + 3) & ~3;
        total = bm + (mins > lists ? mins : lists);
    }
};

// Scratch of one workgroup, in floats: the kept pieces of y, the lists, the
// listed values of each wave, exact group minima.
struct Scratch {
    size_t pool, list, vals, mins, total;
    __host__ __device__ Scratch(int G, bool half, int w, const Dims &d) {
        pool = 64;                                          // reads may start a value early
        list = pool + (size_t)w * d.NG * G + 4 * G;             // and run past the last piece
        list = (list + 63) & ~(size_t)63;
        vals = list + 2 * (size_t)d.nblk * d.items;
        vals = (vals + 63) & ~(size_t)63;
        mins = vals + (size_t)d.NW * d.cap * G;
        mins = (mins + 63) & ~(size_t)63;
        total = mins + (half ? (size_t)w * d.NG + 4 : 0);   // exact group minima [w][NG]
        total = (total + 63) & ~(size_t)63;
    }
};

__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
__device__ __forceinline__ uint32_t key_of(float y) { return __float_as_uint(y); }
__device__ __forceinline__ uint32_t bits(float y) { return __float_as_uint(y); }
__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_min(uint32_t x) {
    return min(x, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)x, CTRL, 0xf, 0xf, false));
}
// Sum over the wave of each lane's predicate.
__device__ __forceinline__ int votes(bool p) { return __popcll(__ballot(p)); }
// Smallest value of the wave (all lanes active), uniform.
__device__ __forceinline__ uint32_t wave_min(uint32_t x) {
    x = dpp_min<0xB1>(x);    // quad_perm [1,0,3,2]
    x = dpp_min<0x4E>(x);    // quad_perm [2,3,0,1]
    x = dpp_min<0x141>(x);   // row_half_mirror
    x = dpp_min<0x140>(x);   // row_mirror
    x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)x, 0x142, 0xa, 0xf, false));  // row_bcast:15
    x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)x, 0x143, 0xc, 0xf, false));  // row_bcast:31
    return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}
__device__ __forceinline__ uint32_t wave_max(uint32_t x) { return ~wave_min(~x); }

__device__ __forceinline__ void exchange(uint32_t &a, uint32_t &b) {  // a <= b afterwards
    const uint32_t x = a, y = b;
    a = min(x, y);
    b = max(x, y);
}
// Sorts a[0..N) ascending (Batcher's odd-even merge network, truncated to N).
template <int N>
__device__ __forceinline__ void sort_net(uint32_t (&a)[N]) {
#pragma unroll
    for (int p = 1; p < N; p += p) {
#pragma unroll
        for (int k = p; k > 0; k /= 2) {
#pragma unroll
            for (int j = k % p; j + k < N; j += 2 * k) {
#pragma unroll
                for (int i = 0; i < k; ++i) {
                    if (i + j + k < N && (i + j) / (2 * p) == (i + j + k) / (2 * p)) exchange(a[i + j], a[i + j + k]);
                }
            }
        }
    }
}
// a[i] for a lane's own 0 <= i < N: a tree of bit selects (an index would make
// the wave loop over its lanes' values).
template <int N>
__device__ __forceinline__ uint32_t pick(const uint32_t (&a)[N], int i) {
    uint32_t t[N];
#pragma unroll
    for (int e = 0; e < N; ++e) t[e] = a[e];
#pragma unroll
    for (int d = 1; d < N; d *= 2) {
        uint32_t odd = i & d ? 0xFFFFFFFFu : 0u;
        asm("" : "+v"(odd));
#pragma unroll
        for (int e = 0; e < N; e += 2 * d)
            if (e + d < N) t[e] = (t[e + d] & odd) | (t[e] & ~odd);
    }
    return t[0];
}

template <int NT_>
__device__ __forceinline__ void stage_f64(double *dst, const double *src, int n, int t, int nt) {
    constexpr int U = NT_;
    for (int b = t; b < n; b += U * nt) {
        double v[U];
#pragma unroll
        for (int e = 0; e < U; ++e) v[e] = b + e * nt < n ? src[b + e * nt] : 0.0;
#pragma unroll
        for (int e = 0; e < U; ++e)
            if (b + e * nt < n) dst[b + e * nt] = v[e];
    }
}

// FP64 anchors of a thread's VA diagonals d0 .. d0+VA-1 of a strip, as in
// pst_profile.hip (the same sums in the same order): the covariance at the
// first cell, (0, d-(w-1)) or (w-1-d, 0).
__device__ __forceinline__ void anchors(float (&cov)[VA], const double *xr, const double *xc, int d0, int w, int l,
                                        const double *mur, const double *muc) {
    const int ub0 = d0 - (w - 1);
    const bool top = ub0 >= 0;
    const int base = -ub0 - (VA - 1);
    const double *P = top ? xr : xc;
    const double *Q = top ? xc + ub0 : xr + base;
    double acc[VA], xs[VA];
#pragma unroll
    for (int v = 0; v < VA; ++v) acc[v] = 0.0;
#pragma unroll
    for (int v = 0; v < VA - 1; ++v) xs[v] = Q[v];
    int tt = 0;
    for (; tt + VA <= l; tt += VA) {
#pragma unroll
        for (int kq = 0; kq < VA; ++kq) {
            xs[(kq + VA - 1) % VA] = Q[tt + kq + VA - 1];
            const double a = P[tt + kq];
#pragma unroll
            for (int v = 0; v < VA; ++v) acc[v] = fma(a, xs[(kq + v) % VA], acc[v]);
        }
    }
    for (; tt < l; ++tt) {
        const double a = P[tt];
#pragma unroll
        for (int v = 0; v < VA; ++v) acc[v] = fma(a, Q[tt + v], acc[v]);
    }
#pragma unroll
    for (int v = 0; v < VA; ++v) {
        const double c = top ? fma(-((double)l * mur[0]), muc[ub0 + v], acc[v])
                             : fma(-((double)l * mur[base + VA - 1 - v]), muc[0], acc[VA - 1 - v]);
        cov[v] = (float)c;
    }
}

// A thread's columns: statistics and the covariance at row 0.
struct Cols {
    float wi[V], wf[V], wg[V], wa[V], cov0[V];
};

// y of one row and the covariance of the next: cov moves one column right,
// the wave's first lane takes the column left of it from `left`.
template <bool CONST>
__device__ __forceinline__ void row_step(const Cols &c, float (&cov)[V], const float4 &r, float left, uint32_t (&y)[V],
                                         float &last) {
    float nx[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const float a = CONST ? c.wa[v] - r.w : c.wa[v];
        y[v] = key_of(__builtin_amdgcn_fmed3f(fmaf(-cov[v] * r.x, c.wi[v], a), 0.0f, 1.0f));
        nx[v] = fmaf(r.y, c.wg[v], fmaf(c.wf[v], r.z, cov[v]));
    }
    last = nx[V - 1];
#pragma unroll
    for (int v = V - 1; v > 0; --v) cov[v] = nx[v - 1];
    // wave_shr:1
    cov[0] = __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(left), __float_as_int(last), 0x138, 0xf, 0xf,
                                                        false));
}

// Minimum of a row over the group of G columns a lane belongs to.
template <int G>
__device__ __forceinline__ uint32_t group_min(const uint32_t (&y)[V]) {
    uint32_t m = min(min(min(y[0], y[1]), y[2]), min(min(y[3], y[4]), y[5]));
    if (G >= 12) m = dpp_min<0xB1>(m);   // quad_perm [1,0,3,2]
    if (G >= 24) m = dpp_min<0x4E>(m);   // quad_perm [2,3,0,1]
    if (G >= 48) m = dpp_min<0x141>(m);  // row_half_mirror
    return m;
}

// First pass: column minima into colmin, group minima into bm, the covariance
// left of each wave into bnd.  Wave k runs a step behind wave k-1.
template <int G, bool H, bool CONST>
__device__ __forceinline__ void pass_one(const Cols &c, uint32_t (&colmin)[V], const float4 *rst, float *bnd, int wp,
                                         uint32_t *bm, uint32_t *gm, int ldg, int NG, int w, int nwa, int wv,
                                         int lane) {
    auto keep = [&](int i, int g, uint32_t m) {
        if constexpr (H) {
            ((uint16_t *)bm)[i * ldg + g] = (uint16_t)(m >> kHalfShift);
            gm[i * NG + g] = m;
        } else {
            bm[i * ldg + g] = m;
        }
    };
    const int nch = (w + RCH - 1) / RCH;
    const int g = (wv * 64 + lane) / (G / V);
    const bool lead = lane % (G / V) == 0 && g < NG;
    const float *lb = bnd + wv * wp;
    float *rb = bnd + (wv + 1) * wp;
    float cov[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
        cov[v] = c.cov0[v];
        colmin[v] = kOne;
    }
    for (int s = 0; s < nch + nwa - 1; ++s) {
        const int ch = s - wv;
        if (wv < nwa && ch >= 0 && ch < nch) {
            const int r0 = ch * RCH;
            if (r0 + RCH <= w) {
                float4 rr[RCH];
                float lf[RCH], out[RCH];
                uint32_t mg[RCH];
#pragma unroll
                for (int e = 0; e < RCH; ++e) {
                    rr[e] = rst[r0 + e];
                    lf[e] = lb[r0 + e + 1];
                }
#pragma unroll
                for (int e = 0; e < RCH; e += 2) {
                    uint32_t y0[V], y1[V];
                    row_step<CONST>(c, cov, rr[e], lf[e], y0, out[e]);
                    row_step<CONST>(c, cov, rr[e + 1], lf[e + 1], y1, out[e + 1]);
#pragma unroll
                    for (int v = 0; v < V; ++v) colmin[v] = min(min(colmin[v], y0[v]), y1[v]);
                    mg[e] = group_min<G>(y0);
                    mg[e + 1] = group_min<G>(y1);
                }
                if (lead) {
#pragma unroll
                    for (int e = 0; e < RCH; ++e) keep(r0 + e, g, mg[e]);
                }
                if (lane == 63 && wv + 1 < nwa) {
#pragma unroll
                    for (int e = 0; e < RCH; ++e) rb[r0 + e + 1] = out[e];
                }
            } else {
                for (int i = r0; i < w; ++i) {
                    uint32_t y[V];
                    float out;
                    row_step<CONST>(c, cov, rst[i], lb[i + 1], y, out);
#pragma unroll
                    for (int v = 0; v < V; ++v) colmin[v] = min(colmin[v], y[v]);
                    const uint32_t m = group_min<G>(y);
                    if (lead) keep(i, g, m);
                    if (lane == 63 && wv + 1 < nwa) rb[i + 1] = out;
                }
            }
        }
        lds_barrier();
    }
}

// Second pass: the pieces of y named in need (16 groups of a row to a word,
// the slots before them in its upper half) into the pool.
template <int G, bool CONST>
__device__ __forceinline__ void pass_two(const Cols &c, const float4 *rst, const float *lb, const uint32_t *need,
                                         int ngw, int NG, float *pool, int w, int t) {
    const int g = t / (G / V);
    const uint32_t bit = g < NG ? 1u << (g & 15) : 0u;
    const uint32_t *nd = need + min(g >> 4, ngw - 1);
    float *mine = pool + (t % (G / V)) * V;
    float cov[V];
#pragma unroll
    for (int v = 0; v < V; ++v) cov[v] = c.cov0[v];
    auto keep = [&](const uint32_t (&y)[V], uint32_t q) {
        if (q & bit) {
            float2 *p = (float2 *)(mine + (size_t)((q >> 16) + __popc(q & (bit - 1u))) * G);
            p[0] = make_float2(__uint_as_float(y[0]), __uint_as_float(y[1]));
            p[1] = make_float2(__uint_as_float(y[2]), __uint_as_float(y[3]));
            p[2] = make_float2(__uint_as_float(y[4]), __uint_as_float(y[5]));
        }
    };
    int i = 0;
    for (; i + RCH <= w; i += RCH) {
        float4 rr[RCH];
        float lf[RCH];
        uint32_t q[RCH];
#pragma unroll
        for (int e = 0; e < RCH; ++e) {
            rr[e] = rst[i + e];
            lf[e] = lb[i + e + 1];
            q[e] = nd[(i + e) * ngw];
        }
#pragma unroll
        for (int e = 0; e < RCH; ++e) {
            uint32_t y[V];
            float out;
            row_step<CONST>(c, cov, rr[e], lf[e], y, out);
            keep(y, q[e]);
        }
    }
    for (; i < w; ++i) {
        uint32_t y[V];
        float out;
        row_step<CONST>(c, cov, rst[i], lb[i + 1], y, out);
        keep(y, nd[i * ngw]);
    }
}

// Keys of the wave that are at most x.
template <int NR>
__device__ __forceinline__ int count_le(const uint32_t (&K)[NR], uint32_t x) {
    int n = 0;
#pragma unroll
    for (int r = 0; r < NR; ++r) n += votes(K[r] <= x);
    return n;
}
// The smallest key above x (signed: -1 is below every key), and the largest
// that is at most x.
template <int NR>
__device__ __forceinline__ uint32_t next_above(const uint32_t (&K)[NR], int x) {
    uint32_t m = kNone;
#pragma unroll
    for (int r = 0; r < NR; ++r) m = min(m, (int)(K[r] & 0x7FFFFFFFu) > x ? K[r] : kNone);
    return wave_min(m);
}
template <int NR>
__device__ __forceinline__ uint32_t last_at(const uint32_t (&K)[NR], uint32_t x) {
    uint32_t m = 0u;
#pragma unroll
    for (int r = 0; r < NR; ++r) m = max(m, K[r] <= x ? K[r] : 0u);
    return wave_max(m);
}

// A point strictly inside (xl, xh), xh - xl > 1, aimed at rank k between the
// counts cl < k <= ch: interpolated, every third time the middle.
__device__ __forceinline__ int aim(int xl, int xh, int cl, int ch, int k, int it) {
    const float d = (float)(xh - xl);
    const float f = it % 3 == 2 ? 0.5f : ((float)(k - cl) - 0.5f) * __builtin_amdgcn_rcpf((float)(ch - cl));
    return min(max(uni(xl + (int)(d * f)), xl + 1), xh - 1);
}

// The k-th smallest of the wave's keys, which lies in (xl, xh] with cl < k
// keys at most xl and ch >= k at most xh.  With slack >= 0 any x at or above it
// that has at most k + slack keys at or below it will do.
template <int NR>
__device__ __forceinline__ uint32_t find_rank(const uint32_t (&K)[NR], int k, int xl, int cl, int xh, int ch,
                                              int slack) {
    for (int it = 0;; ++it) {
        if (slack >= 0 && ch <= k + slack) return (uint32_t)xh;
        if (cl == k - 1 || xh - xl <= 1) return next_above<NR>(K, xl);
        if (ch == k) return last_at<NR>(K, (uint32_t)xh);
        const int x = aim(xl, xh, cl, ch, k, it);
        const int c = count_le<NR>(K, (uint32_t)x);
        if (c >= k) {
            xh = x;
            ch = c;
        } else {
            xl = x;
            cl = c;
        }
    }
}

// The same from a guess x and the spacing of the keys around it: steps that
// double until rank k is bracketed.
template <int NR>
__device__ __forceinline__ uint32_t find_from(const uint32_t (&K)[NR], int k, int x, int step, int most, int xl,
                                              int cl, int top, int slack) {
    int xh = top, ch = 64 * NR;
    x = min(max(x, xl + 1), xh - 1);
    while (x > xl && x < xh) {
        const int c = count_le<NR>(K, (uint32_t)x);
        if (c >= k) {
            xh = x;
            ch = c;
            if (slack >= 0 && ch <= k + slack) return (uint32_t)xh;
            if (cl == k - 1 || ch == k) break;
            if (xl >= 0) break;
            x -= min(step * (c - k + 1), x);   // 0 at the least
        } else {
            xl = x;
            cl = c;
            if (cl == k - 1 || ch != 64 * NR) break;
            x += min(step * (k - c), top);
        }
        step = min(step * 2, most);
    }
    if (ch == 64 * NR) ch = count_le<NR>(K, (uint32_t)xh);
    if (ch < k) return (uint32_t)top;    // fewer than k keys: the largest y there is
    return find_rank<NR>(K, k, xl, cl, xh, ch, slack);
}

// U and C of this lane's rows for block a: the groups a .. a + gc + ge hold the
// columns of the block's windows, a+1 .. a+gc lie inside every one of them.
// GC > 0: gc, GE: ge (fixed loads); GC = 0: any gc >= 4.
template <typename T, int NR, int GC, int GE>
__device__ __forceinline__ void row_keys(uint32_t (&U)[NR], uint32_t (&C)[NR], const T *bm, int ldg, int w, int a,
                                         int lane, int gc, int ge) {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        U[r] = kNone;
        C[r] = kNone;
        if (64 * r < w) {
            const int x = lane + 64 * r;
            if (x < w) {
                const T *row = bm + x * ldg + a;
                uint32_t c = kNone, u;
                if constexpr (GC > 0) {
                    uint32_t m[GC + GE + 1];
#pragma unroll
                    for (int q = 0; q <= GC + GE; ++q) m[q] = row[q];
#pragma unroll
                    for (int q = 1; q <= GC; ++q) c = min(c, m[q]);
                    u = min(c, m[0]);
#pragma unroll
                    for (int q = GC + 1; q <= GC + GE; ++q) u = min(u, m[q]);
                } else {
                    const uint32_t m0 = row[0], e1 = row[gc + 1], e2 = row[gc + ge];
                    for (int q = 0; q < gc; q += 4) {   // the last four overlap the ones before
                        const T *p = row + 1 + min(q, gc - 4);
                        const uint32_t m1 = p[0], m2 = p[1], m3 = p[2], m4 = p[3];
                        c = min(min(min(c, m1), m2), min(m3, m4));
                    }
                    u = min(min(min(c, m0), e1), e2);
                }
                U[r] = u;
                C[r] = c;
            }
        }
    }
}
template <typename T, int NR, int GC0, int GC1>
__device__ __forceinline__ void row_keys_of(uint32_t (&U)[NR], uint32_t (&C)[NR], const T *bm, int ldg, int w, int a,
                                            int lane, int gc, int ge) {
    if constexpr (GC0 < GC1) {
        if (gc > GC0) {
            row_keys_of<T, NR, GC0 + 1, GC1>(U, C, bm, ldg, w, a, lane, gc, ge);
            return;
        }
    }
    if (ge <= 1) row_keys<T, NR, GC0, 1>(U, C, bm, ldg, w, a, lane, gc, ge);
    else row_keys<T, NR, GC0, 2>(U, C, bm, ldg, w, a, lane, gc, ge);
}

// a, b in order.
__device__ __forceinline__ void in_order(uint32_t &a, uint32_t &b) {
    const uint32_t x = min(a, b);
    b = max(a, b);
    a = x;
}
__device__ __forceinline__ void sort8(uint32_t (&s)[8]) {
    constexpr int e[19][2] = {{0, 1}, {2, 3}, {4, 5}, {6, 7}, {0, 2}, {1, 3}, {4, 6}, {5, 7}, {1, 2}, {5, 6},
                              {0, 4}, {3, 7}, {1, 5}, {2, 6}, {1, 4}, {3, 6}, {2, 4}, {3, 5}, {3, 4}};
#pragma unroll
    for (int i = 0; i < 19; ++i) in_order(s[e[i][0]], s[e[i][1]]);
}
// The K smallest of L and S, both in order, in L.
template <int K, int N>
__device__ __forceinline__ void merge_low(uint32_t (&L)[K], const uint32_t (&S)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) L[K - 1 - i] = min(L[K - 1 - i], S[i]);
#pragma unroll
    for (int h = K / 2; h >= 1; h /= 2)
#pragma unroll
        for (int i = 0; i < K; ++i)
            if ((i & h) == 0) in_order(L[i], L[i + h]);
}

// The k-th smallest U (C: the k-th smallest C), k <= K, of nb blocks from a0 at
// once: lane b + nb j takes every parts-th row and column of block a0 + b from
// the j-th on and keeps their K smallest; the parts are merged into lane b.
// A search by counts (find_from) is a chain of ten ballots for one block after
// the other, half of a strip's time at w = 33; keeping K keys in order is 9
// (K = 8) or 14 (K = 16) operations per key with every lane in use: 50 000
// points, w = 33: 7.6 -> 5.5 ms, w = 65: 3.6 -> 3.0.  With K = 32 (groups of 24
// columns) the keys no longer fit the registers: 8.5 -> 9.4 ms at w = 129.
template <int G, int K, bool C>
__device__ __forceinline__ uint32_t block_ranks(int a0, int nb, int parts, int w, int k, int CS, const Dims &d,
                                                const uint32_t *bm, const uint32_t *colk, int lane) {
    const int gc = w / G - 1, ge = 1 + (w - 2) / G - gc;   // as in block_bounds
    const int part = min(lane / nb, parts - 1), a = a0 + lane % nb;
    uint32_t L[K];
#pragma unroll
    for (int i = 0; i < K; ++i) L[i] = part == 0 && i < K - k ? 0u : kNone;
    for (int x0 = part; x0 < w; x0 += 8 * parts) {
        uint32_t s[8];
        int row[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            row[e] = min(x0 + e * parts, w - 1) * d.ldg + a;
            s[e] = bm[row[e] + 1];
            if constexpr (!C) s[e] = min(min(min(bm[row[e]], bm[row[e] + gc + 1]), bm[row[e] + gc + ge]), s[e]);
        }
        for (int q = 2; q <= gc; ++q)
#pragma unroll
            for (int e = 0; e < 8; ++e) s[e] = min(s[e], bm[row[e] + q]);
#pragma unroll
        for (int e = 0; e < 8; ++e) s[e] = x0 + e * parts < w ? s[e] : kNone;
        sort8(s);
        merge_low(L, s);
    }
    const int c1 = C ? w : w + G - 1;
    for (int x0 = part + (C ? G - 1 : 0); x0 < c1; x0 += 8 * parts) {
        uint32_t s[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int cx = x0 + e * parts, cg = a * G + cx;
            const bool on = cx < c1 && cg < CS;
            s[e] = colk[on ? cg : 0];
            s[e] = on ? s[e] : kNone;
        }
        sort8(s);
        merge_low(L, s);
    }
    for (int h = parts / 2; h >= 1; h /= 2) {
        uint32_t o[K];
#pragma unroll
        for (int i = 0; i < K; ++i) o[i] = __shfl(L[i], lane + h * nb);
        merge_low(L, o);
    }
    return min(L[K - 1], kOne);
}

// Bounds and lists of the blocks [a0, a1) of a strip, by one wave; lane + 64 r
// is row i < w or column x - w of the block's columns.  GC0 .. GC1: the whole
// groups inside a block's windows (0: any).  H: the keys are the upper halves,
// rounded down, of the group minima and of the columns alike; a bound lo or hi
// then stands for all keys with that upper half.
template <int G, bool H, int NR, int GC0, int GC1>
__device__ __forceinline__ void block_bounds(int a0, int a1, int w, int k, int CS, const Dims &d, const uint32_t *bm,
                                             const uint32_t *colk, uint32_t *need, uint4 *blk, uint2 *list, int lane) {
    constexpr int SH = H ? kHalfShift : 0;
    constexpr int kTop = (int)(kOne >> SH), kStep0 = H ? 1 : 1 << 10, kStep1 = H ? 64 : 1 << 20;
    const int gc = w / G - 1;                 // groups a+1 .. a+gc lie inside every window of the block
    const int ge = 1 + (w - 2) / G - gc;      // groups past them that hold a column of its windows
    const int rem = w % G;
    uint32_t U[NR], C[NR];
    uint32_t lo = 0x3D800000u >> SH, hi = lo; // guesses: y = 1/16, then the block before
    const bool ranked = G <= 12 && k <= kMaxRank;
    uint32_t los = 0u, his = 0u;
    int from = a0;
    // the pieces that this lane's rows need: bit j is group base + j (one atomic
    // per word and pass over 32 groups instead of three per listed row: w = 33,
    // 6.6 -> 5.5 ms)
    uint32_t nm[NR];
    int base = a0;
#pragma unroll
    for (int r = 0; r < NR; ++r) nm[r] = 0u;
    auto flush = [&]() {
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int x = lane + 64 * r;
            if (64 * r < w && x < w) {
                uint32_t *nd = need + x * d.NGW + (base >> 4);
                const uint64_t q = (uint64_t)nm[r] << (base & 15);
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    const uint32_t p = (uint32_t)(q >> (16 * j)) & 0xFFFFu;
                    if (p) atomicOr(nd + j, p);
                }
                nm[r] = 0u;
            }
        }
    };
    for (int a = a0; a < a1; ++a) {
        if (a - base + w / G + 1 > 31) {
            flush();
            base = a;
        }
        if constexpr (G <= 12) {
            if (ranked && (a - a0) % 64 == 0) {
                from = a;
                const int nb = min(a1 - a, 64), parts = nb > 32 ? 1 : (nb > 16 ? 2 : (nb > 8 ? 4 : 8));
                if (k <= 8) {
                    los = block_ranks<G, 8, false>(a, nb, parts, w, k, CS, d, bm, colk, lane);
                    his = block_ranks<G, 8, true>(a, nb, parts, w, k, CS, d, bm, colk, lane);
                } else {
                    los = block_ranks<G, 16, false>(a, nb, parts, w, k, CS, d, bm, colk, lane);
                    his = block_ranks<G, 16, true>(a, nb, parts, w, k, CS, d, bm, colk, lane);
                }
            }
        }
        if constexpr (H) row_keys<uint16_t, NR, 0, 0>(U, C, (const uint16_t *)bm, d.ldg, w, a, lane, gc, ge);
        else row_keys_of<uint32_t, NR, GC0, GC1>(U, C, bm, d.ldg, w, a, lane, gc, ge);
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            if (64 * r + 63 >= w) {
                const int cx = lane + 64 * r - w, cg = a * G + cx;
                if (cx >= 0 && cx < w + G - 1 && cg < CS) {
                    const uint32_t u = colk[cg] >> SH;
                    U[r] = u;
                    C[r] = cx >= G - 1 && cx < w ? u : kNone;
                }
            }
        }
    // lo: the k-th smallest U; hi: no less than the k-th smallest C
        bool exact;
        if (G <= 12 && ranked) {
            lo = (uint32_t)__builtin_amdgcn_readlane((int)los, a - from);
            hi = (uint32_t)__builtin_amdgcn_readlane((int)his, a - from);
            exact = lo == hi && lo < (uint32_t)kTop;
        } else {
            const int span = max((int)(hi - lo), kStep0), step = min(max(span / 8, kStep0), kStep1);
            lo = find_from<NR>(U, k, (int)lo, step, kStep1, -1, 0, kTop, -1);
            const int ce = count_le<NR>(C, lo);
            if (ce >= k || lo >= (uint32_t)kTop) {
                hi = lo;
            } else {
                hi = find_from<NR>(C, k, (int)max(hi, lo + (uint32_t)span / 2), step, kStep1, (int)lo, ce, kTop,
                                   2 + (k >> 4));
            }
            exact = ce >= k;
        }
        // (an upper half of zero is y = 0 alone: y is a multiple of 2^-50)
        if (exact && (!H || lo == 0u)) {
            if (lane == 0) blk[a] = make_uint4(lo, lo, 0u, 0u);
            continue;
        }
        if constexpr (H) {
            if (exact) {
                int open = 0;
#pragma unroll
                for (int r = 0; r < NR; ++r) open += votes(C[r] >= lo && U[r] <= lo);
                if (open > kOpen) {
                    if (lane == 0) blk[a] = make_uint4(lo, 0u, 0u, kNone);   // for equal_blocks
                    continue;
                }
            }
        }
        // below lo everywhere; listed: the rest that may be at most hi
        int below = 0, n = 0;
        uint2 *la = list + (size_t)a * d.items;
        const int gr = a + w / G;
        const uint32_t bits = (1u | (gr < d.NG ? 1u << (gr - a) : 0u) |
                               (rem >= 2 && gr + 1 < d.NG ? 2u << (gr - a) : 0u)) << (a - base);
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int x = lane + 64 * r;
            const bool b = C[r] < lo;
            const bool in = !b && U[r] <= hi;
            below += votes(b);
            const uint64_t m = __ballot(in);
            if (64 * r < w) nm[r] |= in ? bits : 0u;
            if (m == 0) continue;
            if (in) {
                const int pos = n + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                              __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                const bool isrow = x < w;
                la[pos] = isrow ? make_uint2((uint32_t)x, C[r])
                                : make_uint2(0x80000000u | (uint32_t)(x - w), colk[a * G + x - w]);
            }
            n += __popcll(m);
        }
        if (lane == 0)
            blk[a] = make_uint4(lo << SH, (hi << SH) | ((1u << SH) - 1u), (uint32_t)below, (uint32_t)n);
    }
    flush();
}

// The blocks of half keys that block_bounds left: one upper half holds the k-th
// smallest U and C and more than kOpen items (repeats and constant stretches give
// equal values).  Bounds and list from the whole minima gm of the rows in that
// upper half; those below it count as 0, those above it not at all.  Mostly the
// value is then known, where all those rows' pieces were kept and selected among
// (30 000 points, 40 000 at w = 264, l = m/2, before -> now, k_profile; a quarter of
// a regime series constant: w = 230: 3.0 -> 1.25, 2.4 ms, w = 264: 4.8 -> 1.8, 3.6;
// period 40, with the blocks at y = 0 that block_bounds settles: w = 230: 4.4 ->
// 0.54, 1.9, w = 264: 6.9 -> 0.9, 2.6; a walk of 200 000, w = 257: 43.1 -> 41.3;
// w = 264 with the second workgroup that its CUs hold now).
template <int G, int NR>
__device__ __forceinline__ void equal_blocks(int a0, int a1, int w, int k, int CS, const Dims &d, const uint16_t *bm,
                                             const uint32_t *gm, const uint32_t *colk, uint32_t *need, uint4 *blk,
                                             uint2 *list, int lane) {
    const int gc = w / G - 1, ge = 1 + (w - 2) / G - gc, rem = w % G;   // as in block_bounds
    const int live = min((CS + WCOL - 1) / WCOL * (WCOL / G), d.NG);    // groups that the first pass wrote
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (int a = a0; a < a1; ++a) {
        // opaque, so that no row's address is kept in registers from block to block
        // (89 spilled registers with them, 41 without)
        asm volatile("" : "+v"(lane));
        if (uni((int)blk[a].w) != (int)kNone) continue;
        const uint32_t half = (uint32_t)uni((int)blk[a].x);
        uint32_t U[NR], C[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int x = lane + 64 * r, cx = x - w, cg = a * G + cx;
            U[r] = C[r] = kNone;
            if (x < w) {
                const uint16_t *hb = bm + x * d.ldg + a;
                uint32_t c = kNone;
                for (int q = 1; q <= gc; ++q) c = min(c, (uint32_t)hb[q]);
                const uint32_t u = min(min(c, (uint32_t)hb[0]), min((uint32_t)hb[gc + 1], (uint32_t)hb[gc + ge]));
                if (c < half) {
                    U[r] = C[r] = 0u;
                } else if (u <= half) {
                    const uint32_t *row = gm + x * d.NG + a;
                    c = kNone;
                    for (int q = 1; q <= gc; ++q) c = min(c, row[q]);
                    C[r] = c;
                    U[r] = min(min(c, row[0]), min(row[min(gc + 1, live - 1 - a)], row[min(gc + ge, live - 1 - a)]));
                }
            } else if (cx < w + G - 1 && cg < CS && colk[cg] >> kHalfShift <= half) {
                U[r] = colk[cg];
                if (cx >= G - 1 && cx < w) C[r] = U[r];
            }
        }
        const int under = (int)(half << kHalfShift) - 1, top = under + (1 << kHalfShift);
        const uint32_t lo = find_rank<NR>(U, k, under, count_le<NR>(U, (uint32_t)under), top,
                                          count_le<NR>(U, (uint32_t)top), -1);
        const int cl = count_le<NR>(C, lo);
        if (cl >= k) {
            if (lane == 0) blk[a] = make_uint4(lo, lo, 0u, 0u);
            continue;
        }
        const uint32_t hi = find_rank<NR>(C, k, (int)lo, cl, top, count_le<NR>(C, (uint32_t)top), -1);
        int below = 0, n = 0;
        uint2 *la = list + (size_t)a * d.items;
        const int gr = a + w / G;
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int x = lane + 64 * r;
            const bool b = C[r] < lo, in = !b && U[r] <= hi;
            below += votes(b);
            const uint64_t m = __ballot(in);
            if (in) {
                const int pos = n + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                              __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                if (x < w) {
                    uint32_t *nd = need + x * d.NGW;
                    atomicOr(nd + (a >> 4), 1u << (a & 15));
                    if (gr < d.NG) atomicOr(nd + (gr >> 4), 1u << (gr & 15));
                    if (rem >= 2 && gr + 1 < d.NG) atomicOr(nd + ((gr + 1) >> 4), 1u << ((gr + 1) & 15));
                }
                la[pos] = x < w ? make_uint2((uint32_t)x, C[r]) : make_uint2(0x80000000u | (uint32_t)(x - w), U[r]);
            }
            n += __popcll(m);
        }
        if (lane == 0) blk[a] = make_uint4(lo, hi, (uint32_t)below, (uint32_t)n);
    }
}

// block_bounds with the registers that w needs.
template <int G, bool H, int KR>
__device__ __forceinline__ void strip_bounds(int a0, int a1, int w, int k, int CS, const Dims &d, const uint32_t *bm,
                                             const uint32_t *gm, const uint32_t *colk, uint32_t *need, uint4 *blk,
                                             uint2 *list, int lane) {
    const int nr = (d.items + 63) / 64;
#define BOUNDS(NR, GC0, GC1) block_bounds<G, H, NR, GC0, GC1>(a0, a1, w, k, CS, d, bm, colk, need, blk, list, lane)
    // the widths of each kind: see stream_group and kKindR
    if constexpr (G == 6) {
        BOUNDS(1, 1, 2);
    } else if constexpr (G == 12) {
        if (nr <= 2) BOUNDS(2, 1, 4);
        else BOUNDS(3, 3, 5);
    } else if constexpr (G == 24 && !H) {
        if (nr <= 4) BOUNDS(4, 2, 3);
        else if (nr == 5) BOUNDS(5, 3, 5);
        else BOUNDS(6, 4, 6);
    } else if constexpr (H) {
        if (nr <= 7) BOUNDS(7, 0, 0);
        else BOUNDS(9, 0, 0);
        equal_blocks<G, KR>(a0, a1, w, k, CS, d, (const uint16_t *)bm, gm, colk, need, blk, list, lane);
    } else {
        if (nr <= 13) BOUNDS(13, 4, 7);
        else BOUNDS(18, 6, 10);
    }
#undef BOUNDS
}

// One listed item of block a over the block's G windows, by one lane.
template <int G, bool H>
__device__ __forceinline__ void item_values(uint2 it, int a, int w, const Dims &d, const uint32_t *need,
                                            const float *pool, const uint32_t *gm, uint32_t (&o)[G]) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    typedef f4 f4u __attribute__((aligned(4)));
    if (it.x & 0x80000000u) {  // a column: in the windows that hold it
        const int cx = (int)(it.x & 0x7FFFFFFFu);
#pragma unroll
        for (int p = 0; p < G; ++p) o[p] = (p <= cx && p >= cx - w + 1) ? it.y : kNone;
    } else {
        // a row: suffix minima of its group, the whole groups inside (it.y, or
        // their exact minima gm), and running minima of the columns that follow
        const uint32_t *nd = need + (int)it.x * d.NGW;
        auto slot = [&](int g) {
            const uint32_t q = nd[min(g >> 4, d.NGW - 1)];
            return (int)((q >> 16) + __popc(q & ((1u << (g & 15)) - 1u)));
        };
        const float *pa = pool + (size_t)slot(a) * G;
        const int rem = w % G;
        const float *pr = pool + (size_t)slot(a + w / G) * G;
        const float *pt = pr + rem - 1;
#pragma unroll
        for (int p = 0; p < G; p += 4) {
            const f4 q = *(const f4u *)(pa + p);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (p + e < G) o[p + e] = bits(q[e]);
        }
        uint32_t run = it.y;
        if constexpr (H) {
            typedef uint32_t u4 __attribute__((ext_vector_type(4)));
            typedef u4 u4u __attribute__((aligned(4)));
            const uint32_t *inner = gm + (int)it.x * d.NG + a + 1;
            const int gc = w / G - 1;
            run = kNone;
            for (int q = 0; q < gc; q += 4) {   // the last four overlap the ones before
                const u4 m = *(const u4u *)(inner + min(q, gc - 4));
                run = min(min(min(run, m[0]), m[1]), min(m[2], m[3]));
            }
        }
        for (int x = 0; x < rem - 1; x += 4) {  // columns 0 .. rem-2 (those past it repeat nothing)
            const f4 q = *(const f4u *)(pr + x);
            run = min(run, bits(q[0]));
#pragma unroll
            for (int e = 1; e < 4; ++e) run = min(run, x + e < rem - 1 ? bits(q[e]) : kNone);
        }
#pragma unroll
        for (int p = G - 2; p >= 0; --p) o[p] = min(o[p], o[p + 1]);
        f4 t[(G + 3) / 4];
#pragma unroll
        for (int p = 0; p < (G + 3) / 4; ++p) t[p] = *(const f4u *)(pt + 4 * p);
#pragma unroll
        for (int p = 0; p < G; ++p) {
            const uint32_t y = p == 0 && rem == 0 ? kNone : bits(t[p / 4][p % 4]);
            run = min(run, y);
            o[p] = min(o[p], run);
        }
    }
}

// The kk-th smallest of a window's n <= N listed values, v[e * st] in LDS.
template <int N, int ST>
__device__ __forceinline__ uint32_t select_sorted(const uint32_t *v, int n, int kk) {
    uint32_t c[N];
#pragma unroll
    for (int e = 0; e < N; ++e) c[e] = v[e * ST];
#pragma unroll
    for (int e = 0; e < N; ++e) c[e] = e < n ? c[e] : kNone;
    sort_net(c);
    return pick(c, kk - 1);
}

// As select_sorted for n <= 64 values shared by the lanes p and p + 32: each
// sorts every second one; the 32 smallest of the two lists (or, past rank 32,
// the 32 largest) are the minima (maxima) of one list against the other's
// reverse, and a bitonic merge sorts them.
template <int ST>
__device__ __forceinline__ uint32_t select_halved(const uint32_t *v, int n, int kk, int half) {
    uint32_t c[32], z[32];
    const uint32_t *vh = v + half * ST;
#pragma unroll
    for (int e = 0; e < 32; ++e) c[e] = vh[2 * e * ST];
#pragma unroll
    for (int e = 0; e < 32; ++e) c[e] = 2 * e + half < n ? c[e] : kNone;
    sort_net(c);
    const bool upper = kk > 32;
#pragma unroll
    for (int e = 0; e < 32; ++e) {
        const uint32_t o = (uint32_t)__shfl_xor((int)c[31 - e], 32);
        z[e] = upper ? max(c[e], o) : min(c[e], o);
    }
#pragma unroll
    for (int d = 16; d > 0; d /= 2) {
#pragma unroll
        for (int e = 0; e < 32; ++e)
            if (!(e & d)) exchange(z[e], z[e + d]);
    }
    return pick(z, upper ? kk - 33 : kk - 1);
}

// The kk-th smallest of the wave's n keys: v is a first guess, lo and hi are
// bounds.  A window's value is mostly the one before it or a neighbour in
// rank: two counts, or one reduction more.
template <int NR>
__device__ __forceinline__ uint32_t settle(const uint32_t (&X)[NR], int n, int kk, uint32_t v, uint32_t lo,
                                           uint32_t hi) {
    const int le = count_le<NR>(X, v);
    if (le < kk) {
        if (le == kk - 1) return next_above<NR>(X, (int)v);
        return find_rank<NR>(X, kk, (int)v, le, (int)hi, n, -1);
    }
    int lt = 0;
#pragma unroll
    for (int r = 0; r < NR; ++r) lt += votes(X[r] < v);
    if (lt < kk) return v;
    if (lt == kk) return last_at<NR>(X, v - 1u);
    return find_rank<NR>(X, kk, (int)lo - 1, 0, (int)v - 1, lt, -1);
}

// The values of np windows whose nr * 64 listed values lie at vals[p * 64 nr];
// lane p of the result is window p.
template <int NR>
__device__ __forceinline__ uint32_t select_windows(const uint32_t *vals, int np, int n, int kk, uint32_t &v,
                                                   uint32_t lo, uint32_t hi, int lane) {
    uint32_t res = 0u;
    uint32_t x[NR], nx[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) nx[r] = vals[64 * r + lane];
    for (int p = 0; p < np; ++p) {
#pragma unroll
        for (int r = 0; r < NR; ++r) x[r] = nx[r];
        const uint32_t *next = vals + min(p + 1, np - 1) * (64 * NR) + lane;
#pragma unroll
        for (int r = 0; r < NR; ++r) nx[r] = next[64 * r];
        v = settle<NR>(x, n, kk, v, lo, hi);
        res = lane == p ? v : res;
    }
    return res;
}

struct Strip {
    const ProfileJob *J;
    int s, CS, JSe;     // JSe = 0: only the column minima, for the strip to the left
    int64_t C0;
    const uint32_t *in; // minima of the columns past SBW, from the strip to the right, or null
    uint32_t *out;      // minima of the first w-1 columns, for the strip to the left
};

template <int G, bool H, int KR>
__device__ __forceinline__ void run_strip(const Strip &S, float *sm, float *scr, int NT, int SBW, float &tmax) {
    const ProfileJob &J = *S.J;
    // opaque to the compiler, so that nothing computed from them is kept in
    // registers from one strip to the next
    int w = J.w, t = threadIdx.x;
    asm volatile("" : "+s"(w), "+s"(NT), "+s"(SBW), "+v"(t));
    const int l = J.l;
    const Dims d(G, H, w, NT, SBW);
    const Lds L(H, w, d);
    const Scratch X(G, H, w, d);
    const int wv = uni(t >> 6), lane = t & 63;
    const int64_t rb = (int64_t)S.s * J.row_stride;
    float4 *rst = (float4 *)(sm + L.rst);
    float *bnd = sm + L.bnd;
    float *col = sm + L.col;
    uint32_t *need = (uint32_t *)(sm + L.need);
    uint4 *blk = (uint4 *)(sm + L.blk);
    uint32_t *bm = (uint32_t *)(sm + L.bm);
    uint32_t *gm = (uint32_t *)(scr + X.mins);
    const int CS = S.CS;
    const int nwa = (CS + WCOL - 1) / WCOL;   // waves with columns

    PROBE_MARK(t0);
    // row statistics; the anchors' slices of the centred series
    int crow = 0;
    for (int i = t; i < w; i += NT) {
        const int64_t r = rb + i;
        const float hr = J.row.h[r];
        rst[i] = make_float4(0.5f * J.row.inv[r], J.row.df[r], J.row.dg[r], 0.5f * hr);
        crow |= hr != 0.0f;
    }
    for (int i = t; i < w * d.NGW; i += NT) need[i] = 0u;
    for (int i = CS + t; i < d.NC; i += NT) col[i] = 0.0f;
    const int ndg = CS + w - 1;
    const int off = (VA - (w - 1) % VA) % VA;
    const int ncx = CS + VA + l, nrx = w + l + VA - 2;
    const bool staged = 2 * (ncx + nrx) <= L.total - L.bm;
    double *Xc = (double *)bm, *Xr = Xc + ncx;
    if (staged) {
        stage_f64<4>(Xc, J.col.xc + S.C0, ncx, t, NT);
        stage_f64<4>(Xr, J.row.xc + rb, nrx, t, NT);
    }
    const bool any_const = __syncthreads_or(crow) != 0;
    const int d0 = t * VA - off;
    if (d0 < ndg) {
        float a[VA];
        if (staged) anchors(a, Xr, Xc, d0, w, l, J.row.mu + rb, J.col.mu + S.C0);
        else anchors(a, J.row.xc + rb, J.col.xc + S.C0, d0, w, l, J.row.mu + rb, J.col.mu + S.C0);
#pragma unroll
        for (int v = 0; v < VA; ++v) {
            const int q = d0 + v;
            if (q >= 0 && q < ndg) {
                if (q >= w - 1) col[q - (w - 1)] = a[v];
                else bnd[w - 1 - q] = a[v];
            }
        }
    }
    Cols c;
    const int u0 = t * V;
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int u = u0 + v;
        const bool in = u < CS;
        const int64_t cc = S.C0 + (in ? u : 0);
        // outside the strip: y = 1, neutral for every minimum
        c.wi[v] = in ? J.col.inv[cc] : 0.0f;
        c.wf[v] = in ? J.col.df[cc] : 0.0f;
        c.wg[v] = in ? J.col.dg[cc] : 0.0f;
        c.wa[v] = in ? 0.5f - 0.5f * J.col.h[cc] : 2.0f;
    }
    lds_barrier();
#pragma unroll
    for (int v = 0; v < V; ++v) c.cov0[v] = col[u0 + v];
    uint32_t colmin[V];
    PROBE_SPAN(0, t0);
    PROBE_MARK(t1);
    if (any_const)
        pass_one<G, H, true>(c, colmin, rst, bnd, L.wp, bm, gm, d.ldg, d.NG, w, nwa, wv, lane);
    else
        pass_one<G, H, false>(c, colmin, rst, bnd, L.wp, bm, gm, d.ldg, d.NG, w, nwa, wv, lane);
    uint32_t *colk = (uint32_t *)col;
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int u = u0 + v;
        if (u < w - 1) S.out[u] = colmin[v];
        colk[u] = S.in && u >= SBW && u < CS ? S.in[u - SBW] : colmin[v];
    }
    PROBE_SPAN(1, t1);
    if (S.JSe == 0) return;
    // groups past the last active wave hold nothing
    for (int i = t; i < w; i += NT)
        for (int g = min(nwa * (WCOL / G), d.NG); g <= d.NG; ++g) {
            if constexpr (H) ((uint16_t *)bm)[i * d.ldg + g] = (uint16_t)(kOne >> kHalfShift);
            else bm[i * d.ldg + g] = kOne;
        }
    if constexpr (H) __syncthreads();   // the exact group minima are read by other waves
    else lds_barrier();

    float *pool = scr + X.pool;
    uint2 *list = (uint2 *)(scr + X.list);
    const int nblk = (S.JSe + G - 1) / G;
    const int per = (nblk + d.NW - 1) / d.NW;
    PROBE_MARK(t2);
    strip_bounds<G, H, KR>(min(wv * per, nblk), min(wv * per + per, nblk), w, min(J.k, 2 * w), CS, d, bm, gm, colk,
                           need, blk, list, lane);
    PROBE_SPAN(2, t2);
    __syncthreads();
    PROBE_SPAN(3, t2);
    PROBE_MARK(t3);
    // slots of the kept pieces, in (row, group) order
    if (wv == 0) {
        const int tot = w * d.NGW, pl = (tot + 63) / 64;
        const int b = lane * pl, e = min(b + pl, tot);
        int sum = 0;
        for (int i = b; i < e; ++i) sum += __popc(need[i]);
        int inc = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(inc, o);
            if (lane >= o) inc += y;
        }
        int at = inc - sum;
        for (int i = b; i < e; ++i) {
            const uint32_t q = need[i];
            need[i] = q | (uint32_t)at << 16;
            at += __popc(q);
        }
    }
    lds_barrier();
    if (wv < nwa) {
        const float *lb = bnd + wv * L.wp;
        if (any_const)
            pass_two<G, true>(c, rst, lb, need, d.NGW, d.NG, pool, w, t);
        else
            pass_two<G, false>(c, rst, lb, need, d.NGW, d.NG, pool, w, t);
    }
    __syncthreads();
    PROBE_SPAN(4, t3);
    PROBE_MARK(t4);

    // selection: one lane per listed item for its values over its block, then
    // one lane per window
    const int keff = min(J.k, 2 * w);
    const float four_l = (float)(4 * l);
    uint32_t *lvals = bm + wv * kSelect;   // the group minima are done with
    const int ab = min(wv * per, nblk), ae = min(wv * per + per, nblk);
    auto put = [&](int a, int p, bool on, uint32_t y) {
        if (on) {
            const float dist = sqrtf(four_l * __uint_as_float(y));
            J.D[(int64_t)S.s * J.ld + S.C0 + a * G + p] = dist;
            tmax = fmaxf(tmax, dist);
        }
    };
    auto wave_sync = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    // blocks of up to 32 items are taken several at a time, as many as their
    // windows fit the lanes and their items two (narrow groups) or one a lane
    constexpr int LB = G < 64 ? G : 64, NB = 64 / LB, ST = G + 1;
    constexpr int IT = G <= 12 ? 2 : 1, most = 64 * IT * ST <= kSelect ? 64 * IT : kSelect / ST;   // items of a lane, of a wave
    int cnt = 0, T = 0, nmax = 0;
    int mya = 0, myb = 0;   // of the lane's window: its block, the block's first item
    int ita[IT], itb[IT];   // of the lane's items
#pragma unroll
    for (int h = 0; h < IT; ++h) ita[h] = itb[h] = 0;
    for (int a = ab;; ++a) {
        const bool end = a >= ae;
        const uint4 bl = blk[end ? ab : a];
        const int n0 = end ? 0 : uni((int)bl.w);
        const bool few = n0 > 0 && n0 <= 32;
        if (cnt > 0 && (end || (few && (cnt == NB || T + n0 > most)))) {
            PROBE_MARK(t5);
            PROBE_ADD(8, cnt);
            PROBE_ADD(9, T);
#pragma unroll
            for (int h = 0; h < IT; ++h) {
                const int e = lane + 64 * h;
                if (e < T) {
                    uint32_t o[G];
                    item_values<G, H>(list[(size_t)ita[h] * d.items + (e - itb[h])], ita[h], w, d, need, pool, gm, o);
#pragma unroll
                    for (int p = 0; p < G; ++p) lvals[e * ST + p] = o[p];
                }
            }
            wave_sync();
            PROBE_SPAN(6, t5);
            const int p = lane % LB;
            const bool on = lane / LB < cnt && p < S.JSe - mya * G;
            const uint4 mb = blk[mya];
            const int n = on ? (int)mb.w : 0;
            const uint32_t *v = lvals + (on ? myb * ST + p : 0);
            const int kk = keff - (int)mb.z;
            uint32_t r;
            if (nmax <= 8) r = select_sorted<8, ST>(v, n, kk);
            else if (nmax <= 12) r = select_sorted<12, ST>(v, n, kk);
            else if (nmax <= 16) r = select_sorted<16, ST>(v, n, kk);
            else if (nmax <= 20) r = select_sorted<20, ST>(v, n, kk);
            else if (nmax <= 26) r = select_sorted<26, ST>(v, n, kk);
            else r = select_sorted<32, ST>(v, n, kk);
            put(mya, p, on, r);
            wave_sync();
            cnt = T = nmax = 0;
        }
        if (end) break;
        const int np = min(G, S.JSe - a * G);
        if (n0 == 0) {
            put(a, lane, lane < np, bl.x);
        } else if (few) {
            if (lane / LB >= cnt) {
                mya = a;
                myb = T;
            }
#pragma unroll
            for (int h = 0; h < IT; ++h) {
                if (lane + 64 * h >= T) {
                    ita[h] = a;
                    itb[h] = T;
                }
            }
            ++cnt;
            T += n0;
            nmax = max(nmax, n0);
        } else if (n0 <= 64) {
            PROBE_MARK(t5);
            PROBE_ADD(8, 1);
            PROBE_ADD(9, n0);
            uint32_t o[G];
            item_values<G, H>(list[(size_t)a * d.items + min(lane, n0 - 1)], a, w, d, need, pool, gm, o);
            PROBE_SPAN(6, t5);
            // (the values of gathered blocks, if any, are not in LDS yet)
            constexpr int HW = G < 24 ? G : 24, SH = HW + 1;
#pragma unroll
            for (int h = 0; h < G; h += HW) {
                if (h < np) {
#pragma unroll
                    for (int p = 0; p < HW; ++p) lvals[lane * SH + p] = o[h + p];
                    wave_sync();
                    const int p = lane & 31;
                    const uint32_t r =
                        select_halved<SH>(lvals + min(p, HW - 1), n0, keff - (int)bl.z, lane >> 5);
                    put(a, h + p, lane < HW && h + p < np, r);
                    wave_sync();
                }
            }
        } else if constexpr (KR > 1) {   // more than 64 need as many keys
            PROBE_ADD(8, 1);
            PROBE_ADD(9, n0);
            PROBE_ADD(10, 1);
            PROBE_MARK(t6);
            const int kk = keff - uni((int)bl.z);
            // Two lanes a window, each with half of 64 items at a time: their kKeep
            // smallest (or largest, where that end is the nearer one).  Counts over
            // the wave are some ten steps per window one after the other, four times
            // the time (100 000 points, w = 129: 7.9 -> 7.0 ms, a walk 12.0 -> 8.5).
            // The wider kinds' ranks are further from both ends, and 64 keys a lane
            // leave their registers (w = 257) or are no faster (w = 513).
            const bool up = kk <= kKeep;
            const int kq = up ? kk : n0 - kk + 1;
            if (G == 24 && !H && kq <= kKeep) {
                constexpr int SH = G + 1;
                const int p = min(lane & 31, G - 1);
                uint32_t L[kKeep];
#pragma unroll
                for (int i = 0; i < kKeep; ++i) L[i] = lane < 32 && i < kKeep - kq ? 0u : kNone;
                for (int c0 = 0; c0 < n0; c0 += 64) {
                    uint32_t o[G], c[32];
                    item_values<G, H>(list[(size_t)a * d.items + min(c0 + lane, n0 - 1)], a, w, d, need, pool, gm, o);
#pragma unroll
                    for (int q = 0; q < G; ++q) lvals[lane * SH + q] = c0 + lane < n0 ? (up ? o[q] : ~o[q]) : kNone;
                    wave_sync();
#pragma unroll
                    for (int e = 0; e < 32; ++e) c[e] = lvals[((lane & 32) + e) * SH + p];
                    sort_net(c);
                    merge_low(L, c);
                    wave_sync();
                }
                // the largest of the kKeep smallest of both lanes
                uint32_t r = 0u;
#pragma unroll
                for (int i = 0; i < kKeep; ++i) r = max(r, min(L[i], (uint32_t)__shfl_xor(L[kKeep - 1 - i], 32)));
                put(a, p, lane < np, up ? r : ~r);
                PROBE_SPAN(11, t6);
                continue;
            }
            // (half the kind's keys are fewer than two of each lane at KR = 3)
            constexpr int KH = KR / 2 > 2 ? KR / 2 : 2;
            const int nr = (n0 + 63) / 64, nrr = nr <= 2 ? 2 : (nr <= KH ? KH : KR), stride = 64 * nrr;
            uint32_t *vals = (uint32_t *)(scr + X.vals) + (size_t)wv * d.cap * G;
            for (int e = lane; e < stride; e += 64) {
                uint32_t o[G];
                if (e - lane < n0)
                    item_values<G, H>(list[(size_t)a * d.items + min(e, n0 - 1)], a, w, d, need, pool, gm, o);
#pragma unroll
                for (int p = 0; p < G; ++p) vals[p * stride + e] = e < n0 ? o[p] : kNone;
            }
            // the wave's own stores, read by its other lanes
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
            __builtin_amdgcn_wave_barrier();
            const uint32_t lo = (uint32_t)uni((int)bl.x), hi = (uint32_t)uni((int)bl.y);
            uint32_t v = lo, res;
            if (nrr == 2) res = select_windows<2>(vals, np, n0, kk, v, lo, hi, lane);
            else if (nrr == KH) res = select_windows<KH>(vals, np, n0, kk, v, lo, hi, lane);
            else res = select_windows<KR>(vals, np, n0, kk, v, lo, hi, lane);
            put(a, lane, lane < np, res);
            // the values are read before the next block's are written
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
            __builtin_amdgcn_wave_barrier();
            PROBE_SPAN(11, t6);
        }
    }
    PROBE_SPAN(5, t4);
}

// One run of strips of a job, at = its number among the job's.
template <int G, bool H, int KR>
__device__ __forceinline__ void do_run(const StreamArgs &A, const ProfileJob &J, int64_t at, bool last, float *sm, int NT,
                                       int SBW) {
    const int w = J.w;
    const int ns = (int)((J.Nm + SBW - 1) / SBW);       // strips of a query
    int run = A.run, nrun = (ns + run - 1) / run, s0 = 0;
    if (last && at >= (int64_t)A.tail * nrun) {
        at -= (int64_t)A.tail * nrun;
        s0 = A.tail;
        run = 1;
        nrun = ns;
    }
    const int first = (int)(at % nrun) * run, end = min(first + run, ns);
    uint32_t *carry = (uint32_t *)(sm + Lds(H, w, Dims(G, H, w, NT, SBW)).carry);
    Strip S;
    S.J = &J;
    S.s = s0 + (int)(at / nrun);
    S.in = nullptr;
    float tmax = 0.0f;
    // the strip past the run's end, where the run ends inside a tile
    int i = end < ns && end % A.tile != 0 ? end : end - 1;
    for (; i >= first; --i) {
        S.C0 = (int64_t)i * SBW;
        S.JSe = i < end ? (int)min<int64_t>(SBW, J.Nm - S.C0) : 0;
        S.CS = S.JSe + w - 1;
        S.out = carry + (i & 1) * w;
        __syncthreads();  // the previous strip is done with LDS and the scratch
        run_strip<G, H, KR>(S, sm, J.rw + (size_t)blockIdx.x * A.B.slot_floats, NT, SBW, tmax);
        S.in = i % A.tile != 0 ? S.out : nullptr;
    }
    if (J.dmax_bits) {  // max of D (the denominator of eq. 18): one atomic per wave
        float mx = tmax;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
        if ((threadIdx.x & 63) == 0) atomicMax(J.dmax_bits, __float_as_uint(mx));
    }
}

// Kinds of strip: columns per group, half keys, keys per lane (2w + G - 1 <=
// 64 KR), waves per SIMD.
constexpr int kKindG[kStreamKinds] = {6, 12, 24, 24, 48};
constexpr bool kKindH[kStreamKinds] = {false, false, false, true, false};
constexpr int kKindR[kStreamKinds] = {1, 3, 6, 9, 18};
constexpr int kKindW[kStreamKinds] = {3, 3, 3, 4, 2};
constexpr int kNarrow = 3;   // the first kinds, alike in what a CU holds of them
template <int K>
__host__ __device__ inline int stream_kind_from(int w) {
    if constexpr (K == kStreamKinds) {
        return -1;
    } else {
        constexpr int g = kKindG[K], r = kKindR[K];
        constexpr bool h = kKindH[K];
        return g == stream_group(w) && h == stream_half(w) && 2 * w + g - 1 <= 64 * r ? K : stream_kind_from<K + 1>(w);
    }
}
__host__ __device__ inline int stream_kind(int w) { return stream_kind_from<0>(w); }

// Jobs of the kinds K0 .. K1; NT and LDS are sized for the widest of the launch.
template <int K0, int K1, int WPE>
__global__ void __launch_bounds__(kMaxNT) __attribute__((amdgpu_waves_per_eu(WPE))) k_stream(StreamArgs A) {
    extern __shared__ __align__(16) float sm[];
    __shared__ uint32_t next_run;
    const int NT = blockDim.x, SBW = A.SBW;
    const int64_t total = A.B.tile_end[A.B.njobs - 1];
    int64_t gt = blockIdx.x;
    if (A.B.counter) {
        if (threadIdx.x == 0) next_run = atomicAdd(A.B.counter, 1u);
        __syncthreads();
        gt = next_run;
    }
    while (gt < total) {
        int jb = 0;
        while (jb + 1 < A.B.njobs && gt >= A.B.tile_end[jb]) ++jb;
        const ProfileJob &J = A.B.J[jb];
        const int64_t at = gt - (jb > 0 ? A.B.tile_end[jb - 1] : 0);
        const int kind = K0 == K1 ? K0 : stream_kind(J.w);
        if constexpr (K0 == 0)
            if (kind == 0) do_run<kKindG[0], kKindH[0], kKindR[0]>(A, J, at, jb == A.B.njobs - 1, sm, NT, SBW);
        if constexpr (K0 <= 1 && K1 >= 1)
            if (kind == 1) do_run<kKindG[1], kKindH[1], kKindR[1]>(A, J, at, jb == A.B.njobs - 1, sm, NT, SBW);
        if constexpr (K0 <= 2 && K1 >= 2)
            if (kind == 2) do_run<kKindG[2], kKindH[2], kKindR[2]>(A, J, at, jb == A.B.njobs - 1, sm, NT, SBW);
        if constexpr (K0 <= 3 && K1 >= 3)
            if (kind == 3) do_run<kKindG[3], kKindH[3], kKindR[3]>(A, J, at, jb == A.B.njobs - 1, sm, NT, SBW);
        if constexpr (K1 == 4)
            if (kind == 4) do_run<kKindG[4], kKindH[4], kKindR[4]>(A, J, at, jb == A.B.njobs - 1, sm, NT, SBW);
        if (A.B.counter) {
            __syncthreads();
            if (threadIdx.x == 0) next_run = atomicAdd(A.B.counter, 1u);
            __syncthreads();
            gt = next_run;
        } else {
            gt += gridDim.x;
        }
    }
}

const void *const kKernels[kStreamKinds + 1] = {
    (const void *)k_stream<0, 0, kKindW[0]>, (const void *)k_stream<1, 1, kKindW[1]>,
    (const void *)k_stream<2, 2, kKindW[2]>, (const void *)k_stream<3, 3, kKindW[3]>,
    (const void *)k_stream<4, 4, kKindW[4]>, (const void *)k_stream<0, kNarrow - 1, kKindW[0]>};

// A run of r strips costs 1/r strip's first w-1 columns over again, and ends up
// to r strips after the others: runs as long as leave each workgroup three,
// then four single strips a workgroup (ms, runs to the end / with them: w = 33,
// 50 000 points 5.0 / 4.75; w = 257, a walk of 200 000 45.5 / 43.9; w = 513,
// 100 003 10.4 / 9.8, 200 000 41.4 / 38.6).
constexpr int64_t kRunsPerSlot = 3;
constexpr int64_t kTailStrips = 4;
constexpr size_t kLdsCU = 160 * 1024;
constexpr size_t kLdsStatic = 272;   // next_run and the vote of __syncthreads_or, as compiled
constexpr size_t kLdsUnit = 1280;    // a workgroup's LDS is allocated in these

int stream_threads(int w, int SBW) {
    const int by_col = (SBW + w - 1 + V - 1) / V;
    const int by_diag = (SBW + 2 * w - 2 + VA - 1 + VA - 1) / VA;
    return 64 * ((std::max(by_col, by_diag) + 63) / 64);
}

}  // namespace

size_t stream_lds_bytes(int32_t w, int32_t wmax, int32_t SBW) {
    const bool H = stream_half(w);
    return 4 * (size_t)Lds(H, w, Dims(stream_group(w), H, w, stream_threads(wmax, SBW), SBW)).total;
}

// k_profile keeps the windows that hold no two groups of six columns.  From
// there to w = 552 this kernel is the better one at the default rank (ms, l =
// m/2, k_profile against it; 50 000 points of a regime series / a random walk):
// w = 12: 14.6 / 14.3 against 8.7 / 8.6, w = 17: 16.2 / 16.0 against 7.7 / 7.7,
// w = 24: 14.0 / 13.8 against 5.5 / 5.4, w = 33: 6.4 / 5.7 against 4.9 / 5.1,
// w = 65: 4.2 / 4.7 against 2.9 / 3.8; 5 000 points: w = 12: 0.51 against 0.20,
// w = 33: 0.45 against 0.13.  w = 552 is where a block's rows and columns fill
// kKindR = 18 keys a lane.
bool stream_takes(int32_t w, int32_t SBW) {
    if (w < 12 || stream_kind(w) < 0) return false;
    return stream_threads(w, SBW) <= kMaxNT && stream_lds_bytes(w, w, SBW) + kLdsStatic <= kLdsCU;
}

// Ranks at which this kernel is the better one in a launch that fills the chip
// either way.  Towards the middle of a window's 2w values the bounds leave most
// rows open, the more so the wider a group is against w, while k_profile's time
// hardly depends on k.  Time of this kernel over k_profile's, 50 000 and 60 000
// points, the worse of a regime series and a random walk / white noise, on both
// sides of each line: w = 17: k = 16 0.8 / 0.9, 17 1.4 / 1.5; w = 33: k = 10
// 0.96 / 1.0, 13 1.02 / 1.2, 33 1.8 / 2.2; w = 47: k = 16 0.9 / 0.9, 19 1.3 / 1.4;
// w = 65: k = 26 1.03 / 1.1, 49 1.14 / 1.4; w = 90: k = 54 0.95 / 1.2, 68 1.08 /
// 1.4; w = 265: k = 133 0.98 / 1.3, 265 1.2 / 1.5.  The largest value (k = 2w) is
// cheap again but at w = 265 .. 289 and 32 .. 35.  w = 24 .. 31: 0.3 .. 0.8 at
// every rank (a walk's), 144 .. 264 and 290 on: 1.0 at the most, 1.3 in noise.
bool stream_ranks(int32_t w, int32_t k) {
    if (k >= 2 * w) return w < 32 || (w >= 36 && w < 265) || w >= 290;
    if (w < 24) return k <= kMaxRank;
    if (w < 32) return true;
    if (w < 36) return k <= w / 3;
    if (w < 48) return k <= kMaxRank;
    if (w < 80) return 5 * k <= 2 * w;
    if (w < 144) return 5 * k <= 3 * w;
    if (w >= 265 && w < 290) return 2 * k <= w;
    return true;
}

size_t stream_slot_floats(int32_t w, int32_t wmax, int32_t SBW) {
    const int G = stream_group(w);
    const bool H = stream_half(w);
    return Scratch(G, H, w, Dims(G, H, w, stream_threads(wmax, SBW), SBW)).total;
}

// Workgroups resident at once: LDS and the registers' waves, as the runtime counts
// them at every w.  (With 512 bytes for the static LDS the plan left w = 264 one
// workgroup a CU of two and w = 144 three of four: 60 000 points, l = w - 1, 4.9 ->
// 3.0 and 2.8 -> 2.3 ms.)
int32_t stream_slots(int32_t w, int32_t SBW) {
    const int NT = stream_threads(w, SBW);
    const size_t units = (stream_lds_bytes(w, w, SBW) + kLdsStatic + kLdsUnit - 1) / kLdsUnit;
    const size_t by_lds = kLdsCU / (kLdsUnit * units);
    const size_t by_waves = 4 * kKindW[stream_kind(w)] / (NT / 64);
    return 256 * (int32_t)std::max<size_t>(1, std::min(by_lds, by_waves));
}

// Workgroups of the kernel of w resident on a CU, by the runtime.
hipError_t stream_occupancy(int32_t w, int32_t SBW, int *per_cu) {
    const hipError_t e = stream_prepare();
    if (e != hipSuccess) return e;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, kKernels[stream_kind(w)], stream_threads(w, SBW),
                                                        stream_lds_bytes(w, w, SBW));
}

hipError_t stream_prepare() {
    for (const void *k : kKernels) {
        const hipError_t e =
            hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(kLdsCU - kLdsStatic));
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_stream(const ProfileJob *jobs, int n, int32_t SBW, int32_t tile, size_t scratch_floats,
                         double share, int32_t limit, uint32_t *counter, hipStream_t st) {
    if (n < 1 || n > kMaxJobs) return hipErrorInvalidValue;
    int kinds = 0;
    for (int i = 0; i < n; ++i) {
        if (!stream_takes(jobs[i].w, SBW)) return hipErrorInvalidValue;
        kinds |= 1 << stream_kind(jobs[i].w);
    }
    // One launch per kind among the jobs, widest first.  The narrow kinds share
    // one: each launch ends with a strip's latency on a chip that empties (lengths
    // 64, 80 .. 176, 5 000 points, w = 33 .. 89: 1.5 ms in two, 0.9 in one).  The
    // wider ones hold other numbers of waves: all kinds in one kernel at two waves
    // per SIMD take 7.0 ms where separate launches take 5.2 (96, 128 .. 320,
    // 20 000 points).
    const int narrow = kinds & ((1 << kNarrow) - 1);
    const bool mixed = (narrow & (narrow - 1)) != 0;
    for (int kind = kStreamKinds - 1; kind >= 0; --kind) {
        const bool all = mixed && kind == kNarrow - 1;
        const int set = all ? narrow : (mixed && kind < kNarrow ? 0 : kinds & 1 << kind);
        if (set == 0) continue;
        StreamArgs a;
        a.SBW = SBW;
        a.B.njobs = 0;
        a.B.counter = counter ? counter + kind : nullptr;
        a.B.slot_floats = 0;
        int32_t wmax = 0;
        int64_t strips = 0;
        for (int i = 0; i < n; ++i)
            if (set >> stream_kind(jobs[i].w) & 1) {
                wmax = std::max(wmax, jobs[i].w);
                strips += ((jobs[i].Nm + SBW - 1) / SBW) * (int64_t)jobs[i].nq;
            }
        size_t lds = 0;
        for (int i = 0; i < n; ++i)
            if (set >> stream_kind(jobs[i].w) & 1) {
                a.B.slot_floats = std::max(a.B.slot_floats, stream_slot_floats(jobs[i].w, wmax, SBW));
                lds = std::max(lds, stream_lds_bytes(jobs[i].w, wmax, SBW));
            }
        if (lds + kLdsStatic > kLdsCU) return hipErrorInvalidValue;
        const int32_t slots = stream_slots(wmax, SBW);
        const int64_t most = limit > 0 ? std::min(limit, slots) : std::max<int64_t>(1, (int64_t)(share * slots));
        a.tile = tile;
        a.run = tile;
        while (a.run > 1 && (a.run % 2 != 0 || strips < kRunsPerSlot * most * a.run)) a.run = a.run % 2 ? 1 : a.run / 2;
        int64_t acc = 0;
        for (int k = kStreamKinds - 1; k >= 0; --k)
            for (int i = 0; i < n; ++i) {
                if (stream_kind(jobs[i].w) != k || !(set >> k & 1)) continue;
                const int j = a.B.njobs++;
                a.B.J[j] = jobs[i];
                const int64_t ns = (jobs[i].Nm + SBW - 1) / SBW;
                acc += ((ns + a.run - 1) / a.run) * (int64_t)jobs[i].nq;
                a.B.tile_end[j] = acc;
                a.tail = jobs[i].nq;
            }
        if (a.run > 1) {   // the launch ends with single strips, some for every workgroup
            const ProfileJob &J = a.B.J[a.B.njobs - 1];
            const int64_t ns = (J.Nm + SBW - 1) / SBW;
            a.tail = (int32_t)std::max<int64_t>(0, J.nq - (kTailStrips * most + ns - 1) / ns);
            acc += (J.nq - a.tail) * (ns - (ns + a.run - 1) / a.run);
            a.B.tile_end[a.B.njobs - 1] = acc;
        }
        const int64_t fit = (int64_t)(scratch_floats / a.B.slot_floats);
        const int64_t grid = std::min(std::min(acc, fit), most);
        if (grid < 1) return hipErrorInvalidValue;
        void *args[] = {&a};
        const hipError_t e = hipLaunchKernel(kKernels[all ? kStreamKinds : kind], dim3((unsigned)grid),
                                             dim3(stream_threads(wmax, SBW)), args, lds, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace pst

#ifdef PST_PROBE
// Sums since the last reset: wave cycles of 0 setup and anchors, 1 the first
// pass, 2 bounds, 3 bounds and their barrier, 4 the second pass, 5 selection,
// 6 the listed rows' minima in it, 11 selections of long lists in it; 8 blocks,
// 9 listed items, 10 blocks with long lists.
extern "C" int pst_stream_probe_read(unsigned long long *out, int reset) {
    static unsigned long long buf[16 * 64];
    if (hipMemcpyFromSymbol(buf, HIP_SYMBOL(g_stream_probe), sizeof(buf)) != hipSuccess) return -3;
    for (int i = 0; i < 16; ++i) {
        out[i] = 0;
        for (int j = 0; j < 64; ++j) out[i] += buf[i * 64 + j];
    }
    if (reset) {
        static const unsigned long long zero[16 * 64] = {};
        if (hipMemcpyToSymbol(HIP_SYMBOL(g_stream_probe), zero, sizeof(zero)) != hipSuccess) return -3;
    }
    return 0;
}
#endif
