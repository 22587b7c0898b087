// bjacobi.hip -- block-Jacobi preconditioner (Sec. 3.2): batched in-place
// Gauss-Jordan inversion of the diagonal blocks (4 to 64 blocks a wave),
// adaptive storage precision of each inverse (binary16/32/64 chosen from
// the block's condition number and exponent range), the product z = M r,
// and the CG steps that use it (the r update fused with z = M r and the
// r.z, r.r reductions).
//
// Uniform blocks are consecutive ranges of BS rows (BS in {1,...,32}, the
// last one may be shorter), so a 256-row tile always holds whole blocks.
// Every inverse is stored as a BS x BS row-major array (zeros outside a
// short last block) at byte offset off[b] (a multiple of 16) in the
// precision prec[b].
//
// Variable-size blocks (at most 32 rows each, boundaries given or found by
// supervariable agglomeration) are inverted by the same elimination: blocks
// are sorted into classes by the power of two that holds them and each class
// runs the kernel of that width on a list of its blocks.  Block b's m x m
// inverse is stored row by row, each row padded to whole 16-byte chunks.
// A block reaches at most 31 rows beyond a 256-row tile, so the products
// stage the tile's vector part with 31 rows on either side in LDS.
#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <type_traits>
#include <vector>

#include "device_common.hpp"
#include "internal.hpp"

namespace mxl {

enum { BJ_P64 = 0, BJ_P32 = 1, BJ_P16 = 2 };

// Nearest-even rounding to binary16 from the format's definition: 11-bit
// significand, exponents -14..15, subnormal quantum 2^-24, overflow to
// infinity from 65520 on.  Scaling by the quantum is exact, rint rounds to
// nearest even.
__device__ __forceinline__ double round_f16(double x) {
    if (x == 0.0 || !__builtin_isfinite(x)) return x;
    const double a = fabs(x);
    if (a >= 65520.0) return copysign(__builtin_inf(), x);
    int e2;
    (void)frexp(a, &e2);
    int e = e2 - 1;
    if (e < -14) e = -14;
    const double quantum = ldexp(1.0, e - 10);
    return copysign(rint(a / quantum) * quantum, x);
}

// Rows of the block in slot `slot` of a launch: uniform blocks are slots
// themselves (b = slot, rows b*BS ..); with variable sizes the slot indexes
// a list of block ids of one size class and bptr gives the rows.
struct BlockSel {
    const int *list;      // variable sizes: block ids of this launch's class
    const int *bptr;      // variable sizes: block boundaries
    const int64_t *toff;  // variable sizes: offset of block b's m x m inverse in the output
    int64_t every;        // uniform: slot s is block s * every
};

template <int BS, bool VAR>
__device__ __forceinline__ void block_rows(int64_t slot, int64_t n, const BlockSel &sel, int64_t &b, int64_t &r0,
                                           int &m) {
    if constexpr (VAR) {
        b = sel.list[slot];
        r0 = sel.bptr[b];
        m = sel.bptr[b + 1] - (int)r0;
    } else {
        b = slot * sel.every;
        r0 = b * BS;
        m = (int)(n - r0 < BS ? n - r0 : BS);
    }
}

// Where the inverses of a launch go.  Variable sizes: inv, m x m at toff, FP64
// rounded to the block's precision.  Uniform: inv, BS x BS at b, not rounded; or
// packed into store, block b at b * stride, on the assumption that all blocks
// take the precision `want`; or, with neither, nowhere (a look at the
// precisions).  A block that takes another one sets *mixed, and workgroups that
// start later leave at once.
struct BlockOut {
    double *inv;
    unsigned char *store;
    int64_t stride;
    int want;
    int *mixed;
    int *redo;  // set if a step met an infinity or NaN: the result is to be had from the strict variant
};

// Bytes of a uniform block's inverse: padded to 16 (vector row loads).
__host__ __device__ constexpr int64_t bj_stride(int bs, int prec) {
    return ((int64_t)bs * bs * (prec == BJ_P16 ? 2 : prec == BJ_P32 ? 4 : 8) + 15) / 16 * 16;
}

// Lane l's value (l a constant) within every group of LPB lanes.
template <int LPB, typename T>
__device__ __forceinline__ T group_lane(T v, int l) {
    static_assert(LPB == 1 || LPB == 2 || LPB == 4 || LPB == 8 || LPB == 16, "");
    typedef typename std::conditional<sizeof(T) == 8, long long, int>::type U;
    U u;
    __builtin_memcpy(&u, &v, sizeof u);
#define MXL_BC16(N) case N: u = __builtin_amdgcn_update_dpp((U)0, u, 0x150 + N, 0xf, 0xf, true); break;
#define MXL_BC8(N)                                                                        \
    case N: {                                                                             \
        const U w = __builtin_amdgcn_update_dpp((U)0, u, 0x150 + N, 0xf, 0xf, true);      \
        u = __builtin_amdgcn_update_dpp(w, u, 0x158 + N, 0xf, 0xc, false);                \
        break;                                                                            \
    }
    if constexpr (LPB == 16) {
        switch (l) {
            MXL_BC16(0) MXL_BC16(1) MXL_BC16(2) MXL_BC16(3) MXL_BC16(4) MXL_BC16(5) MXL_BC16(6) MXL_BC16(7)
            MXL_BC16(8) MXL_BC16(9) MXL_BC16(10) MXL_BC16(11) MXL_BC16(12) MXL_BC16(13) MXL_BC16(14) MXL_BC16(15)
        }
    } else if constexpr (LPB == 8) {
        switch (l) {
            MXL_BC8(0) MXL_BC8(1) MXL_BC8(2) MXL_BC8(3) MXL_BC8(4) MXL_BC8(5) MXL_BC8(6) MXL_BC8(7)
        }
    } else if constexpr (LPB > 1) {
        v = __shfl(v, (int)(threadIdx.x % kWave) / LPB * LPB + l, kWave);
        return v;
    }
#undef MXL_BC8
#undef MXL_BC16
    __builtin_memcpy(&v, &u, sizeof u);
    return v;
}

template <int LPB, typename T>
__device__ __forceinline__ T group_max(T v) {
#pragma unroll
    for (int off = LPB / 2; off > 0; off >>= 1) {
        T o = __shfl_xor(v, off, kWave);
        v = o > v ? o : v;
    }
    return v;
}

// binary16 of a double that is zero or within its normal range, nearest even.
__device__ __forceinline__ _Float16 narrow_f16(double x) {
    unsigned long long u = (unsigned long long)__double_as_longlong(x);
    u += ((1ull << 41) - 1) + ((u >> 42) & 1);
    u &= ~((1ull << 42) - 1);
    return (_Float16)(float)(x == x ? __longlong_as_double((long long)u) : x);
}

// One wave inverts P diagonal blocks, one per group of LPB lanes, in place:
// lane l of a group holds S columns of its block in registers (col = S*l + s;
// the block is staged through LDS once, 16 rows at a time, to turn rows into
// columns), and step c turns column c of the block into the column of the
// inverse that belongs to row c's original row (rows are swapped by partial
// pivoting).  Column c's entries reach the group by a lane broadcast inside the
// vector unit, so a step is vector arithmetic with no barrier.  Every element of the
// inverse sees the same operations in the same order as a sequential
// Gauss-Jordan elimination of (D | I) with partial pivoting (first row of
// largest magnitude), with no multiply-add contraction, so the inverse, its
// condition number and the precision decision are reproducible.  (A zero may
// differ in its sign: where the sequential elimination skips a row with a zero
// entry, -0 minus a product of -0 becomes +0 here.)
//
// Bound by vector instructions (busy 68% of the cycles at two waves a SIMD; D is
// 128 registers, and what stands beside it at 32 rows exceeds the other 128 by
// 180 to 200 bytes of scratch a lane): 2 of FP64 per element and step and a
// broadcast per row.
// 128,000 blocks of 32: 4.4 ms with D and I side by side, one block a wave and
// scalar broadcasts -> 1.05 ms.
//
// A zero entry times a finite row changes nothing, so the rows are updated
// without looking at their entries: branches or selects cost more than the
// arithmetic.  Where a row holds an infinity or a NaN the sequential
// elimination skips zero entries all the same; STRICT does that, and the other
// variant only reports the case.
template <int BS, bool VAR, bool STRICT>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(2))) void k_bj_invert(int64_t n, const int *__restrict__ rp,
                                                     const int *__restrict__ col,
                                                     const double *__restrict__ val, int adaptive,
                                                     double accuracy, double *__restrict__ cond,
                                                     int *__restrict__ prec, int *__restrict__ bad, BlockSel sel,
                                                     int64_t nslots, BlockOut out) {
#pragma clang fp contract(off)
    constexpr int LPB = BS < 16 ? BS : 16, S = BS / LPB, P = kWave / LPB;
    __shared__ double L[P][LPB][BS + 1];
    const int lane = threadIdx.x, q = lane / LPB, l = lane % LPB;
    const int64_t slot = (int64_t)blockIdx.x * P + q;
    if (!VAR && !out.inv && __hip_atomic_load(out.mixed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
    const bool live = slot < nslots;
    int64_t b = 0, r0 = 0;
    int m = 0;
    if (live) block_rows<BS, VAR>(slot, n, sel, b, r0, m);
    double D[S][BS];
    int id[S];  // original row of row S*l + s; of column S*l + s once it is eliminated
#pragma unroll
    for (int h = 0; h < S; ++h) {  // rows h*LPB ..: lane l loads row h*LPB + l
#pragma unroll
        for (int e = lane; e < P * LPB * BS; e += kWave) L[e / (LPB * BS)][(e / BS) % LPB][e % BS] = 0.0;
        __syncthreads();
        const int i = h * LPB + l;
        if (i < m) {
            const int k1 = rp[r0 + i + 1];
            for (int k = rp[r0 + i]; k < k1; k += 4) {
                int c[4];
                double v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int ku = k + u < k1 ? k + u : k1 - 1;
                    c[u] = col[ku];
                    v[u] = val[ku];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int64_t cu = (int64_t)c[u] - r0;
                    if (k + u < k1 && cu >= 0 && cu < m) L[q][l][cu] = v[u];
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int i2 = 0; i2 < LPB; ++i2)
#pragma unroll
            for (int s = 0; s < S; ++s) D[s][h * LPB + i2] = L[q][i2][S * l + s];
        __syncthreads();
    }
#pragma unroll
    for (int s = 0; s < S; ++s) id[s] = S * l + s;
    // rows and columns past a short last block hold zeros, which change no sum,
    // maximum or pivot
    auto norm1 = [&]() {
        double best = 0.0;
#pragma unroll
        for (int s = 0; s < S; ++s) {
            double t = 0.0;
#pragma unroll
            for (int i = 0; i < BS; ++i) t += fabs(D[s][i]);
            best = t > best || t != t ? t : best;  // a NaN stays, as in a lane of its own
        }
        return group_max<LPB>(best);
    };
    const double nD = norm1();
    bool singular = false, odd = false;
#pragma clang loop unroll(full)
    for (int c = 0; c < BS; ++c) {
        const int cl = c / S, cs = c % S;  // the lane and slot of column c
        const bool mine = l == cl;
        // the diagonal is the pivot unless something below it is larger
        // (a NaN never is)
        double below = 0.0;
#pragma clang loop unroll(full)
        for (int i = c + 1; i < BS; ++i) below = __builtin_fmax(below, fabs(D[cs][i]));
        const double dcc = fabs(D[cs][c]);
        if (__builtin_expect(__any(mine && c < m && !singular && !(dcc > 0.0 && !(below > dcc))), 0)) {
            // pivot: the first row i >= c of largest |D[i][c]|
            const double best = __builtin_fmax(below, dcc);
            int pv = c;
#pragma clang loop unroll(full)
            for (int i = BS - 1; i >= c; --i) pv = fabs(D[cs][i]) == best ? i : pv;
            const double mx = group_lane<LPB>(best, cl);
            const int piv = group_lane<LPB>(pv, cl);
            if (!singular && c < m && !(mx > 0.0)) singular = true;  // zero column below the diagonal
            if (!singular && c < m && piv != c) {
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    const double dc = D[s][c];
#pragma clang loop unroll(full)
                    for (int i = c + 1; i < BS; ++i)
                        if (i == piv) {
                            asm volatile("");
                            D[s][c] = D[s][i];
                            D[s][i] = dc;
                        }
                }
            }
            int idp = 0;  // rows c and piv trade names
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const int t = __shfl(id[s], q * LPB + piv / S, kWave);
                if (piv % S == s) idp = t;
            }
            const int idc = group_lane<LPB>(id[cs], cl);
            if (!singular && c < m) {
                if (mine) id[cs] = idp;
#pragma unroll
                for (int s = 0; s < S; ++s)
                    if (piv != c && S * l + s == piv) id[s] = idc;
            }
        }
        const bool act = !singular && c < m;
        const double d = group_lane<LPB>(D[cs][c], cl);
        double row[S];  // row c of the result; column c starts from the identity
#pragma unroll
        for (int s = 0; s < S; ++s) row[s] = (s == cs && mine ? 1.0 : D[s][c]) / d;
        if constexpr (!STRICT) {
#pragma unroll
            for (int s = 0; s < S; ++s) {
                odd = odd || (act && !__builtin_isfinite(row[s]));
                row[s] = act ? row[s] : 0.0;
            }
        }
        constexpr int G = BS < 8 ? BS : 8;  // broadcasts ahead of their use
#pragma clang loop unroll(full)
        for (int g = 0; g < BS; g += G) {
            double f[G];
#pragma clang loop unroll(full)
            for (int r = g; r < g + G; ++r) f[r - g] = group_lane<LPB>(D[cs][r], cl);
            if (act && mine) {
                asm volatile("");  // stays a branch: selects would cost as much as the update
#pragma clang loop unroll(full)
                for (int r = g; r < g + G; ++r)
                    if (r != c) D[cs][r] = 0.0;
            }
#pragma clang loop unroll(full)
            for (int r = g; r < g + G; ++r) {
                if (r == c || (STRICT && (!act || f[r - g] == 0.0))) continue;
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    const double pd = f[r - g] * row[s];
                    D[s][r] = D[s][r] - pd;
                }
            }
        }
#pragma unroll
        for (int s = 0; s < S; ++s) D[s][c] = act ? row[s] : D[s][c];
    }
    if (!STRICT && __any(odd)) {
        if (lane == 0) *out.redo = 1;
        return;
    }
    if (singular && l == 0) atomicMin(bad, (int)(b < INT_MAX ? b : INT_MAX));
    const double nI = norm1();
    const double kappa = nD * nI;
    int p = BJ_P64;
    if (adaptive) {
        double lo = __builtin_inf(), hi = 0.0;
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int i = 0; i < BS; ++i) {
                const double a = fabs(D[s][i]);
                lo = __builtin_fmin(lo, a == 0.0 ? lo : a);
                hi = __builtin_fmax(hi, a);
            }
        lo = -group_max<LPB>(-lo);
        hi = group_max<LPB>(hi);
        if (hi == 0.0) lo = hi = 1.0;
        if (kappa * ldexp(1.0, -11) <= accuracy && lo >= ldexp(1.0, -14) && hi <= 65504.0) p = BJ_P16;
        else if (kappa * ldexp(1.0, -24) <= accuracy && lo >= ldexp(1.0, -126) && hi <= 3.4028234663852886e38)
            p = BJ_P32;
    }
    p = group_lane<LPB>(p, 0);  // lanes differ if the block holds a NaN
    if (!live || singular) return;
    if (l == 0) {
        cond[b] = kappa;
        prec[b] = p;
    }
    if constexpr (VAR) {
#pragma unroll
        for (int i = 0; i < BS; ++i)
#pragma unroll
            for (int s = 0; s < S; ++s) {
                double x = D[s][i];
                if (p == BJ_P32) x = (double)(float)x;
                else if (p == BJ_P16) x = round_f16(x);
                if (i < m && S * l + s < m) out.inv[sel.toff[b] + (int64_t)i * m + id[s]] = x;
            }
    } else {
        if (!out.inv && p != out.want) {
            if (l == 0) *out.mixed = 1;
            return;
        }
        if (!out.inv && !out.store) return;
        const bool whole = m == BS;
        bool in_place = S > 1;
#pragma unroll
        for (int s = 0; s < S; ++s) in_place = in_place && id[s] == S * l + s;
        in_place = __all(in_place);
        auto put = [&](auto *o, auto narrow) {
            typedef decltype(narrow(0.0)) T;
            typedef T TS __attribute__((ext_vector_type(S == 1 ? 2 : S)));
#pragma unroll
            for (int i = 0; i < BS; ++i) {
                T t[S];
#pragma unroll
                for (int s = 0; s < S; ++s)  // zeros outside a short last block
                    t[s] = narrow(whole || (i < m && S * l + s < m) ? D[s][i] : 0.0);
                if constexpr (S > 1) {
                    if (in_place) {
                        TS w;
#pragma unroll
                        for (int s = 0; s < S; ++s) w[s] = t[s];
                        *(TS *)(o + i * BS + S * l) = w;
                        continue;
                    }
                }
#pragma unroll
                for (int s = 0; s < S; ++s) o[i * BS + id[s]] = t[s];
            }
        };
        unsigned char *base = out.store + b * out.stride;
        if (out.inv) put(out.inv + b * BS * BS, [](double x) { return x; });
        else if (p == BJ_P16) put((_Float16 *)base, [](double x) { return narrow_f16(x); });
        else put((double *)base, [](double x) { return x; });
    }
}

// Offsets of blocks of mixed precisions: the exclusive sums of their sizes, and
// the total.  Workgroup g owns blocks [g * chunk, (g + 1) * chunk): the first
// kernel sums every chunk, the second adds the sums before its own and scans it
// kScanWG blocks at a time.
constexpr int kScanWG = 1024, kScanGrid = 256;

__device__ __forceinline__ int64_t scan_wg(int64_t v, int64_t &all) {  // inclusive sum over the workgroup
    __shared__ int64_t part[kScanWG / kWave];
    const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
    for (int o = 1; o < kWave; o <<= 1) {
        const int64_t u = __shfl_up(v, o, kWave);
        if (lane >= o) v += u;
    }
    if (lane == kWave - 1) part[wid] = v;
    __syncthreads();
    all = 0;
    for (int w = 0; w < kScanWG / kWave; ++w) {
        v += w < wid ? part[w] : 0;
        all += part[w];
    }
    __syncthreads();
    return v;
}

__global__ __launch_bounds__(kScanWG) void k_bj_sizes(int64_t nb, int64_t chunk, int bs, const int *__restrict__ prec,
                                                      int64_t *__restrict__ sums) {
    const int64_t b0 = blockIdx.x * chunk, b1 = b0 + chunk < nb ? b0 + chunk : nb;
    int64_t v = 0, all;
    for (int64_t b = b0 + threadIdx.x; b < b1; b += kScanWG) v += bj_stride(bs, prec[b]);
    (void)scan_wg(v, all);
    if (threadIdx.x == 0) sums[blockIdx.x] = all;
}

__global__ __launch_bounds__(kScanWG) void k_bj_scan(int64_t nb, int64_t chunk, int bs, const int *__restrict__ prec,
                                                     const int64_t *__restrict__ sums, int64_t *__restrict__ off,
                                                     int64_t *__restrict__ total) {
    const int64_t b0 = blockIdx.x * chunk, b1 = b0 + chunk < nb ? b0 + chunk : nb;
    int64_t base, all;
    (void)scan_wg(threadIdx.x < blockIdx.x ? sums[threadIdx.x] : 0, base);
    for (int64_t t = b0; t < b1; t += kScanWG) {
        const int64_t b = t + threadIdx.x;
        const int64_t sz = b < b1 ? bj_stride(bs, prec[b]) : 0;
        const int64_t v = scan_wg(sz, all);
        if (b < b1) off[b] = base + v - sz;
        base += all;
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *total = base;
}

// Offsets of blocks of one size.
__global__ void k_bj_offsets(int64_t nb, int64_t stride, int64_t *__restrict__ off) {
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b < nb) off[b] = b * stride;
}

// Rounds inverses of mixed precisions into their storage (what takes binary16
// lies in its normal range).
template <int BS>
__global__ void k_bj_pack(int64_t nb, const double *__restrict__ inv, const int *__restrict__ prec,
                          const int64_t *__restrict__ off, unsigned char *__restrict__ store) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= nb * BS * BS) return;
    const int64_t b = e / (BS * BS), k = e % (BS * BS);
    unsigned char *base = store + off[b];
    const double x = inv[e];
    switch (prec[b]) {
    case BJ_P16: ((_Float16 *)base)[k] = narrow_f16(x); break;
    case BJ_P32: ((float *)base)[k] = (float)x; break;
    default: ((double *)base)[k] = x; break;
    }
}

// Row t of block b's stored inverse times the block's vector part held in
// LDS (xs[0..BS)), summed over ascending columns in FP64.  Blocks start at
// 16-byte-aligned offsets, so a row whose bytes are a multiple of 16 is
// read with 16-byte vector loads (8 binary16, 4 binary32 or 2 binary64
// values each); other rows element by element.
template <typename T, int BS>
__device__ __forceinline__ double bj_row_t(const unsigned char *__restrict__ base, int t, const double *xs) {
    constexpr int E = 16 / (int)sizeof(T);
    double s = 0.0;
    if constexpr (BS * sizeof(T) % 16 == 0) {
        typedef T TV __attribute__((ext_vector_type(E)));
        const TV *rp = (const TV *)base + t * (BS / E);
#pragma unroll
        for (int c = 0; c < BS / E; ++c) {
            const TV v = rp[c];
#pragma unroll
            for (int e = 0; e < E; ++e) s += (double)v[e] * xs[c * E + e];
        }
    } else {
        const T *rp = (const T *)base + t * BS;
#pragma unroll
        for (int j = 0; j < BS; ++j) s += (double)rp[j] * xs[j];
    }
    return s;
}

template <int BS>
__device__ __forceinline__ double bj_row(const unsigned char *__restrict__ store, int64_t off, int pr,
                                         int t, const double *xs) {
    const unsigned char *base = store + off;
    if (pr == BJ_P16) return bj_row_t<_Float16, BS>(base, t, xs);
    if (pr == BJ_P32) return bj_row_t<float, BS>(base, t, xs);
    return bj_row_t<double, BS>(base, t, xs);
}

// z = M r on 256-row tiles (whole blocks): each wave parks its 64 values of
// r in LDS, then lane l forms row (l mod BS) of its block.
#define MXL_BJ_TILE(n)                                                  \
    const int L = blockIdx.x;                                           \
    int64_t tb_, te_;                                                   \
    int ts_;                                                            \
    band_walk(((n) + kWG - 1) / kWG, blockIdx.x, gridDim.x, tb_, te_, ts_);

template <int BS>
__global__ __launch_bounds__(kWG) void k_bj_apply(int64_t n, const unsigned char *__restrict__ store,
                                                  const int64_t *__restrict__ off,
                                                  const int *__restrict__ prec, double alpha,
                                                  const double *__restrict__ r, double beta,
                                                  double *__restrict__ z, const int *stop) {
    if (stop && *stop) return;  // inside a solve: nothing after a device-side stop uses z
    __shared__ double xs[kWG];
    MXL_BJ_TILE(n)
    (void)L;
    const int lane = threadIdx.x;
    for (int64_t t_ = tb_; t_ < te_; t_ += ts_) {
        const int64_t i = t_ * kWG + lane;
        xs[lane] = i < n ? r[i] : 0.0;
        __syncthreads();
        if (i < n) {
            const int64_t blk = i / BS;
            const int t = (int)(i % BS);
            const double v = bj_row<BS>(store, off[blk], prec[blk], t, xs + (lane - t));
            z[i] = beta == 0.0 ? alpha * v : alpha * v + beta * z[i];
        }
        __syncthreads();
    }
}

// CG with block Jacobi, initial step: z = M r, p = z; publishes [r.z, r.r, b.b].
// V is the vector type: with binary32 vectors z is rounded to binary32
// before it enters p and r.z (the inverses are still applied in FP64).
template <typename V, int BS>
__global__ __launch_bounds__(kWG) void k_cg_init_bj(int64_t n, const V *__restrict__ b,
                                                    const V *__restrict__ r, V *__restrict__ p,
                                                    const unsigned char *__restrict__ store,
                                                    const int64_t *__restrict__ off,
                                                    const int *__restrict__ prec,
                                                    double *__restrict__ parts) {
    __shared__ double xs[kWG];
    MXL_BJ_TILE(n)
    const int lane = threadIdx.x;
    double rz = 0.0, rr = 0.0, bb = 0.0;
    for (int64_t t_ = tb_; t_ < te_; t_ += ts_) {
        const int64_t i = t_ * kWG + lane;
        const double ri = i < n ? (double)r[i] : 0.0;
        xs[lane] = ri;
        __syncthreads();
        if (i < n) {
            const int64_t blk = i / BS;
            const int t = (int)(i % BS);
            const V zv = (V)bj_row<BS>(store, off[blk], prec[blk], t, xs + (lane - t));
            p[i] = zv;
            rz += ri * (double)zv;
            rr += ri * ri;
            bb += (double)b[i] * (double)b[i];
        }
        __syncthreads();
    }
    double v[3] = {rz, rr, bb};
    publish<3>(v, parts, L);
}

// CG with block Jacobi, after the fused p.q: alpha = rho_{k-1} / p.q,
// r -= alpha q (in FP64, rounded to V), z = M r (rounded to V), and the
// reductions r.z, r.r.  The stop handshake with k_cg_pupdate (st->ustop) is
// the one of the point-Jacobi kernels.
template <typename V, int BS>
__global__ __launch_bounds__(kWG) void k_cg_update_bj(int64_t n, V *__restrict__ r,
                                                      const V *__restrict__ q, V *__restrict__ z,
                                                      const unsigned char *__restrict__ store,
                                                      const int64_t *__restrict__ off,
                                                      const int *__restrict__ prec, SolverState *st,
                                                      const double *__restrict__ pq_parts, int pq_slots,
                                                      double *__restrict__ parts, int k) {
    __shared__ double xs[kWG];
    if (st->stop) {
        if (blockIdx.x == 0 && threadIdx.x == 0) st->ustop = 1;
        return;
    }
    double eta[1];
    gather_all<1>(pq_parts, pq_slots, eta);
    const bool chk = st->nonfinite_check != 0;
    const bool nonfin = chk && !finite_d(eta[0]);
    if (nonfin || eta[0] <= 0.0) {
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            st->stop = nonfin ? ST_NONFINITE : ST_BREAKDOWN;
            st->ustop = 1;
            st->iters = k - 1;
            st->eta = eta[0];
        }
        return;
    }
    const double alpha = st->rho2[(k - 1) & 1] / eta[0];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st->alpha = alpha;
        st->eta = eta[0];
        st->ustop = 0;
    }
    MXL_BJ_TILE(n)
    const int lane = threadIdx.x;
    double rz = 0.0, rr = 0.0;
    for (int64_t t_ = tb_; t_ < te_; t_ += ts_) {
        const int64_t i = t_ * kWG + lane;
        double ri = 0.0;
        if (i < n) {
            V rv;
            if constexpr (sizeof(V) == 8) rv = r[i] - alpha * q[i];
            else rv = (V)((double)r[i] - alpha * (double)q[i]);
            r[i] = rv;
            ri = (double)rv;
        }
        xs[lane] = ri;
        __syncthreads();
        if (i < n) {
            const int64_t blk = i / BS;
            const int t = (int)(i % BS);
            const V zv = (V)bj_row<BS>(store, off[blk], prec[blk], t, xs + (lane - t));
            z[i] = zv;
            rz += ri * (double)zv;
            rr += ri * ri;
        }
        __syncthreads();
    }
    double v[2] = {rz, rr};
    publish<2>(v, parts, L);
}

// ------------------------------------------------ variable-size blocks
constexpr int kBjMax = 32;            // largest block
constexpr int kBjHalo = kBjMax - 1;   // rows a block can reach beyond a tile
constexpr int kBjWin = kWG + 2 * kBjHalo;

// same[i] = 1 when row i has exactly the column set of row i - 1 (a
// supervariable continues), 0 otherwise (same[0] = 0).
__global__ void k_bj_same_prev(int64_t n, const int *__restrict__ rp, const int *__restrict__ col,
                               unsigned char *__restrict__ same) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    unsigned char f = 0;
    if (i > 0) {
        const int a0 = rp[i - 1], a1 = rp[i], b1 = rp[i + 1];
        if (a1 - a0 == b1 - a1) {
            f = 1;
            for (int k = 0; k < a1 - a0; ++k)
                if (col[a0 + k] != col[a1 + k]) {
                    f = 0;
                    break;
                }
        }
    }
    same[i] = f;
}

// rblk[i] = b for every row of block b (one thread per block).
__global__ void k_bj_rowmap(int64_t nb, const int *__restrict__ bptr, int *__restrict__ rblk) {
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= nb) return;
    for (int i = bptr[b]; i < bptr[b + 1]; ++i) rblk[i] = (int)b;
}

// 16-byte chunks per stored row of an m-wide block in precision pr.
__host__ __device__ __forceinline__ int bjv_chunks(int m, int pr) {
    const int e = pr == BJ_P16 ? 8 : pr == BJ_P32 ? 4 : 2;
    return (m + e - 1) / e;
}

// Packs block b's m x m inverse (FP64, already rounded to its precision)
// into rows of whole 16-byte chunks, padding with zeros; one workgroup per
// block.
__global__ void k_bj_pack_var(int64_t nb, const int *__restrict__ bptr, const int64_t *__restrict__ toff,
                              const double *__restrict__ inv, const int *__restrict__ prec,
                              const int64_t *__restrict__ off, unsigned char *__restrict__ store) {
    const int64_t b = blockIdx.x;
    if (b >= nb) return;
    const int m = bptr[b + 1] - bptr[b], pr = prec[b];
    const int ld = bjv_chunks(m, pr) * (pr == BJ_P16 ? 8 : pr == BJ_P32 ? 4 : 2);
    unsigned char *base = store + off[b];
    for (int e = threadIdx.x; e < m * ld; e += blockDim.x) {
        const int i = e / ld, j = e % ld;
        const double x = j < m ? inv[toff[b] + (int64_t)i * m + j] : 0.0;
        switch (pr) {
        case BJ_P16: ((_Float16 *)base)[e] = (_Float16)x; break;
        case BJ_P32: ((float *)base)[e] = (float)x; break;
        default: ((double *)base)[e] = x; break;
        }
    }
}

// Row t of an m-wide stored inverse times xs[0..m), ascending columns, FP64;
// 16-byte loads, the padding lanes of the last chunk are not multiplied (a
// neighbouring row's Inf or NaN must not reach this row).
template <typename T>
__device__ __forceinline__ double bjv_row_t(const unsigned char *__restrict__ base, int t, int m,
                                            const double *xs) {
    constexpr int E = 16 / (int)sizeof(T);
    typedef T TV __attribute__((ext_vector_type(E)));
    const int nv = (m + E - 1) / E;
    const TV *rowp = (const TV *)base + (int64_t)t * nv;
    double s = 0.0;
    for (int c = 0; c < nv; ++c) {
        const TV v = rowp[c];
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (c * E + e < m) s += (double)v[e] * xs[c * E + e];
    }
    return s;
}

__device__ __forceinline__ double bjv_row(const unsigned char *__restrict__ store, int64_t off, int pr, int t,
                                          int m, const double *xs) {
    const unsigned char *base = store + off;
    if (pr == BJ_P16) return bjv_row_t<_Float16>(base, t, m, xs);
    if (pr == BJ_P32) return bjv_row_t<float>(base, t, m, xs);
    return bjv_row_t<double>(base, t, m, xs);
}

// Block row of row i (inside the tile starting at t0) against the staged
// window xw = rows t0 - kBjHalo .. t0 + kWG + kBjHalo.
__device__ __forceinline__ double bjv_apply_row(int64_t i, int64_t t0, const int *__restrict__ rblk,
                                                const int *__restrict__ bptr,
                                                const unsigned char *__restrict__ store,
                                                const int64_t *__restrict__ off, const int *__restrict__ prec,
                                                const double *xw) {
    const int b = rblk[i];
    const int r0 = bptr[b], m = bptr[b + 1] - r0;
    return bjv_row(store, off[b], prec[b], (int)(i - r0), m, xw + (r0 - (t0 - kBjHalo)));
}

// z = alpha M r + beta z with variable-size blocks.
__global__ __launch_bounds__(kWG) void k_bj_apply_var(int64_t n, const int *__restrict__ rblk,
                                                      const int *__restrict__ bptr,
                                                      const unsigned char *__restrict__ store,
                                                      const int64_t *__restrict__ off,
                                                      const int *__restrict__ prec, double alpha,
                                                      const double *__restrict__ r, double beta,
                                                      double *__restrict__ z, const int *stop) {
    if (stop && *stop) return;
    __shared__ double xw[kBjWin];
    MXL_BJ_TILE(n)
    (void)L;
    const int lane = threadIdx.x;
    for (int64_t t_ = tb_; t_ < te_; t_ += ts_) {
        const int64_t t0 = t_ * kWG;
        for (int w = lane; w < kBjWin; w += kWG) {
            const int64_t row = t0 - kBjHalo + w;
            xw[w] = row >= 0 && row < n ? r[row] : 0.0;
        }
        __syncthreads();
        const int64_t i = t0 + lane;
        if (i < n) {
            const double v = bjv_apply_row(i, t0, rblk, bptr, store, off, prec, xw);
            z[i] = beta == 0.0 ? alpha * v : alpha * v + beta * z[i];
        }
        __syncthreads();
    }
}

// CG initial step with variable-size blocks: z = M r, p = z; publishes
// [r.z, r.r, b.b] (as k_cg_init_bj).
template <typename V>
__global__ __launch_bounds__(kWG) void k_cg_init_bjv(int64_t n, const V *__restrict__ b,
                                                     const V *__restrict__ r, V *__restrict__ p,
                                                     const int *__restrict__ rblk, const int *__restrict__ bptr,
                                                     const unsigned char *__restrict__ store,
                                                     const int64_t *__restrict__ off,
                                                     const int *__restrict__ prec, double *__restrict__ parts) {
    __shared__ double xw[kBjWin];
    MXL_BJ_TILE(n)
    const int lane = threadIdx.x;
    double rz = 0.0, rr = 0.0, bb = 0.0;
    for (int64_t t_ = tb_; t_ < te_; t_ += ts_) {
        const int64_t t0 = t_ * kWG;
        for (int w = lane; w < kBjWin; w += kWG) {
            const int64_t row = t0 - kBjHalo + w;
            xw[w] = row >= 0 && row < n ? (double)r[row] : 0.0;
        }
        __syncthreads();
        const int64_t i = t0 + lane;
        if (i < n) {
            const double ri = xw[lane + kBjHalo];
            const V zv = (V)bjv_apply_row(i, t0, rblk, bptr, store, off, prec, xw);
            p[i] = zv;
            rz += ri * (double)zv;
            rr += ri * ri;
            bb += (double)b[i] * (double)b[i];
        }
        __syncthreads();
    }
    double v[3] = {rz, rr, bb};
    publish<3>(v, parts, L);
}

// CG update with variable-size blocks: as k_cg_update_bj, but r_out =
// r_in - alpha q goes to a second buffer, because each workgroup also forms
// the new residual of the 31 rows on either side of its tile (the rows its
// blocks reach into) from r_in, which its neighbours must not overwrite.
template <typename V>
__global__ __launch_bounds__(kWG) void k_cg_update_bjv(int64_t n, const V *__restrict__ r_in,
                                                       V *__restrict__ r_out, const V *__restrict__ q,
                                                       V *__restrict__ z, const int *__restrict__ rblk,
                                                       const int *__restrict__ bptr,
                                                       const unsigned char *__restrict__ store,
                                                       const int64_t *__restrict__ off,
                                                       const int *__restrict__ prec, SolverState *st,
                                                       const double *__restrict__ pq_parts, int pq_slots,
                                                       double *__restrict__ parts, int k) {
    __shared__ double xw[kBjWin];
    if (st->stop) {
        if (blockIdx.x == 0 && threadIdx.x == 0) st->ustop = 1;
        return;
    }
    double eta[1];
    gather_all<1>(pq_parts, pq_slots, eta);
    const bool chk = st->nonfinite_check != 0;
    const bool nonfin = chk && !finite_d(eta[0]);
    if (nonfin || eta[0] <= 0.0) {
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            st->stop = nonfin ? ST_NONFINITE : ST_BREAKDOWN;
            st->ustop = 1;
            st->iters = k - 1;
            st->eta = eta[0];
        }
        return;
    }
    const double alpha = st->rho2[(k - 1) & 1] / eta[0];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st->alpha = alpha;
        st->eta = eta[0];
        st->ustop = 0;
    }
    MXL_BJ_TILE(n)
    const int lane = threadIdx.x;
    double rz = 0.0, rr = 0.0;
    for (int64_t t_ = tb_; t_ < te_; t_ += ts_) {
        const int64_t t0 = t_ * kWG;
        for (int w = lane; w < kBjWin; w += kWG) {
            const int64_t row = t0 - kBjHalo + w;
            double rv = 0.0;
            if (row >= 0 && row < n) {
                V v;
                if constexpr (sizeof(V) == 8) v = r_in[row] - alpha * q[row];
                else v = (V)((double)r_in[row] - alpha * (double)q[row]);
                rv = (double)v;
                if (w >= kBjHalo && w < kBjHalo + kWG) r_out[row] = v;
            }
            xw[w] = rv;
        }
        __syncthreads();
        const int64_t i = t0 + lane;
        if (i < n) {
            const double ri = xw[lane + kBjHalo];
            const V zv = (V)bjv_apply_row(i, t0, rblk, bptr, store, off, prec, xw);
            z[i] = zv;
            rz += ri * (double)zv;
            rr += ri * ri;
        }
        __syncthreads();
    }
    double v[2] = {rz, rr};
    publish<2>(v, parts, L);
}

// ------------------------------------------------------------ host side
#define MXL_BS_SWITCH(BSV, ...)                      \
    switch (BSV) {                                   \
    case 1: { constexpr int BS = 1; __VA_ARGS__; } break;   \
    case 2: { constexpr int BS = 2; __VA_ARGS__; } break;   \
    case 4: { constexpr int BS = 4; __VA_ARGS__; } break;   \
    case 8: { constexpr int BS = 8; __VA_ARGS__; } break;   \
    case 16: { constexpr int BS = 16; __VA_ARGS__; } break; \
    case 32: { constexpr int BS = 32; __VA_ARGS__; } break; \
    default: return hipErrorInvalidValue;            \
    }

hipError_t bj_cg_init(const mxl_ctx *ctx, const JacobiImpl &P, int dtype, int64_t n, const void *b,
                      const void *r, void *p, double *parts, hipStream_t s) {
    const int g = vec_grid(ctx, n);
    const unsigned char *store = (const unsigned char *)P.bstore->p;
    const int64_t *off = (const int64_t *)P.boff->p;
    const int *prec = (const int *)P.bprec->p;
    if (P.var) {
        const int *rb = (const int *)P.rblk->p, *bp = (const int *)P.bptr_d->p;
        if (dtype == MXL_F32)
            hipLaunchKernelGGL(k_cg_init_bjv<float>, dim3(g), dim3(kWG), 0, s, n, (const float *)b,
                               (const float *)r, (float *)p, rb, bp, store, off, prec, parts);
        else
            hipLaunchKernelGGL(k_cg_init_bjv<double>, dim3(g), dim3(kWG), 0, s, n, (const double *)b,
                               (const double *)r, (double *)p, rb, bp, store, off, prec, parts);
        return hipGetLastError();
    }
    if (dtype == MXL_F32) {
        MXL_BS_SWITCH(P.bs, hipLaunchKernelGGL((k_cg_init_bj<float, BS>), dim3(g), dim3(kWG), 0, s, n,
                                               (const float *)b, (const float *)r, (float *)p, store, off,
                                               prec, parts));
    } else {
        MXL_BS_SWITCH(P.bs, hipLaunchKernelGGL((k_cg_init_bj<double, BS>), dim3(g), dim3(kWG), 0, s, n,
                                               (const double *)b, (const double *)r, (double *)p, store, off,
                                               prec, parts));
    }
    return hipGetLastError();
}

hipError_t bj_cg_update(const mxl_ctx *ctx, const JacobiImpl &P, int dtype, int64_t n, const void *r_in,
                        void *r_out, const void *q, void *z, SolverState *st, const double *pq_parts, int pq_slots,
                        double *parts, int k, hipStream_t s) {
    const int g = vec_grid(ctx, n);
    const unsigned char *store = (const unsigned char *)P.bstore->p;
    const int64_t *off = (const int64_t *)P.boff->p;
    const int *prec = (const int *)P.bprec->p;
    if (P.var) {
        if (r_in == r_out) return hipErrorInvalidValue;
        const int *rb = (const int *)P.rblk->p, *bp = (const int *)P.bptr_d->p;
        if (dtype == MXL_F32)
            hipLaunchKernelGGL(k_cg_update_bjv<float>, dim3(g), dim3(kWG), 0, s, n, (const float *)r_in,
                               (float *)r_out, (const float *)q, (float *)z, rb, bp, store, off, prec, st, pq_parts,
                               pq_slots, parts, k);
        else
            hipLaunchKernelGGL(k_cg_update_bjv<double>, dim3(g), dim3(kWG), 0, s, n, (const double *)r_in,
                               (double *)r_out, (const double *)q, (double *)z, rb, bp, store, off, prec, st,
                               pq_parts, pq_slots, parts, k);
        return hipGetLastError();
    }
    if (r_in != r_out) return hipErrorInvalidValue;
    void *r = r_out;
    if (dtype == MXL_F32) {
        MXL_BS_SWITCH(P.bs, hipLaunchKernelGGL((k_cg_update_bj<float, BS>), dim3(g), dim3(kWG), 0, s, n,
                                               (float *)r, (const float *)q, (float *)z, store, off, prec, st,
                                               pq_parts, pq_slots, parts, k));
    } else {
        MXL_BS_SWITCH(P.bs, hipLaunchKernelGGL((k_cg_update_bj<double, BS>), dim3(g), dim3(kWG), 0, s, n,
                                               (double *)r, (const double *)q, (double *)z, store, off, prec,
                                               st, pq_parts, pq_slots, parts, k));
    }
    return hipGetLastError();
}

hipError_t bj_apply(const mxl_ctx *ctx, const JacobiImpl &P, int64_t n, double alpha, const void *r,
                    double beta, void *z, hipStream_t s, const int *stop) {
    const int g = vec_grid(ctx, n);
    if (P.var) {
        hipLaunchKernelGGL(k_bj_apply_var, dim3(g), dim3(kWG), 0, s, n, (const int *)P.rblk->p,
                           (const int *)P.bptr_d->p, (const unsigned char *)P.bstore->p, (const int64_t *)P.boff->p,
                           (const int *)P.bprec->p, alpha, (const double *)r, beta, (double *)z, stop);
        return hipGetLastError();
    }
    MXL_BS_SWITCH(P.bs, hipLaunchKernelGGL(k_bj_apply<BS>, dim3(g), dim3(kWG), 0, s, n,
                                           (const unsigned char *)P.bstore->p, (const int64_t *)P.boff->p,
                                           (const int *)P.bprec->p, alpha, (const double *)r, beta,
                                           (double *)z, stop));
    return hipGetLastError();
}

static hipError_t bj_invert(const MatrixImpl &A, int bs, int adaptive, double accuracy, double *cond, int *prec,
                            int *bad, const BlockOut &out, bool strict, int64_t nb, int64_t every, hipStream_t s) {
    const BlockSel none{nullptr, nullptr, nullptr, every};
    const int per = kWave / (bs < 16 ? bs : 16);  // blocks of a wave
    const dim3 g((unsigned)((nb + per - 1) / per));
    const int *rp = (const int *)A.row_ptr->p, *col = (const int *)A.col->p;
    const double *val = (const double *)A.val->p;
    if (strict) {
        MXL_BS_SWITCH(bs, hipLaunchKernelGGL((k_bj_invert<BS, false, true>), g, dim3(kWave), 0, s, A.nrows, rp, col, val,
                                             adaptive, accuracy, cond, prec, bad, none, nb, out));
    } else {
        MXL_BS_SWITCH(bs, hipLaunchKernelGGL((k_bj_invert<BS, false, false>), g, dim3(kWave), 0, s, A.nrows, rp, col, val,
                                             adaptive, accuracy, cond, prec, bad, none, nb, out));
    }
    return hipGetLastError();
}

static hipError_t bj_pack(int bs, int64_t nb, const double *inv, const int *prec, const int64_t *off,
                          unsigned char *store, hipStream_t s) {
    const int64_t total = nb * bs * bs;
    const unsigned g = (unsigned)((total + 255) / 256);
    MXL_BS_SWITCH(bs, hipLaunchKernelGGL(k_bj_pack<BS>, dim3(g), dim3(256), 0, s, nb, inv, prec, off, store));
    return hipGetLastError();
}

}  // namespace mxl

using namespace mxl;

extern "C" mxl_status mxl_bjacobi_generate(const mxl_op *Aop, int32_t block_size, int32_t adaptive,
                                           double accuracy, mxl_op **Pout) try {
    if (!Aop || !Pout || Aop->kind != MXL_OP_MATRIX)
        return set_error(MXL_ERR_INVALID_ARG, "matrix operator and output required");
    *Pout = nullptr;
    const auto &A = Aop->mat;
    if (block_size != 1 && block_size != 2 && block_size != 4 && block_size != 8 && block_size != 16 &&
        block_size != 32)
        return set_error(MXL_ERR_INVALID_ARG, "block_size must be 1, 2, 4, 8, 16 or 32");
    if (A->nrows != A->ncols) return set_error(MXL_ERR_NOT_IMPLEMENTED, "block Jacobi needs a square matrix");
    if (A->dtype != MXL_F64) return set_error(MXL_ERR_NOT_IMPLEMENTED, "block Jacobi needs an FP64 matrix");
    if (A->format == MXL_FMT_STENCIL)
        return set_error(MXL_ERR_NOT_IMPLEMENTED, "block Jacobi needs stored matrix rows");
    if (A->nrows == 0) return set_error(MXL_ERR_INVALID_ARG, "empty matrix");
    if (!(accuracy >= 0.0)) return set_error(MXL_ERR_INVALID_ARG, "accuracy must be >= 0");
    if (accuracy == 0.0) accuracy = 0.1;
    DeviceScope ds(A->ctx->device);
    hipStream_t s = A->ctx->stream;
    const int bs = block_size;
    const int64_t nb = (A->nrows + bs - 1) / bs;
    auto J = std::make_shared<JacobiImpl>();
    J->A = A;
    J->block = true;
    J->bs = bs;
    J->nblocks = nb;
    // One precision for all blocks is the common outcome (binary16 for blocks
    // worth preconditioning with, binary64 without the adaptive choice): the
    // inverses are packed where they will stay on that assumption.  The first
    // block that takes another precision ends that pass; the inverses then go
    // through a binary64 copy, as their places follow from all precisions.  Without
    // the copy 128,000 blocks of 32 take 0.26 GB of new memory instead of 1.3 GB.
    // A large storage is not allocated before some blocks have been looked at:
    // that costs about 50 us, allocating and freeing it in vain 300.  Below 16 MB
    // the copy is taken at once; a failed guess costs more than the copy does
    // (mixed precisions: 27,000 blocks of 8 took 752 us with it and take 151,
    // 2,000 blocks of 32 took 778 and take 186).
    Arena ar;
    BufPtr flags;
    ar.want(J->bcond, (size_t)nb * 8);
    ar.want(J->boff, (size_t)nb * 8);
    ar.want(J->bprec, (size_t)nb * 4);
    // What a pass leaves for the host, then the sums of the offsets' chunks.
    struct Flags {
        int bad, mixed, redo, pad;  // lowest singular block, whether precisions differ, whether to invert strictly
        int64_t total;              // bytes of the storage, where the pass found the offsets
    } hf;
    ar.want(flags, sizeof(Flags) + kScanGrid * 8);
    auto mk = [&](int64_t bytes) {
        auto d = std::make_shared<DevBuf>();
        if (hipMalloc(&d->p, (size_t)bytes) != hipSuccess) return BufPtr();
        d->bytes = (size_t)bytes;
        d->owned = true;
        return d;
    };
    BlockOut out{};
    out.want = adaptive ? BJ_P16 : BJ_P64;
    out.stride = bj_stride(bs, out.want);
    if (!ar.alloc()) return set_error(MXL_ERR_OUT_OF_MEMORY, "block Jacobi workspace");
    auto *fl = (Flags *)flags->p;
    int *prec = (int *)J->bprec->p;
    int64_t *off = (int64_t *)J->boff->p, *sums = (int64_t *)(fl + 1);
    out.mixed = &fl->mixed;
    out.redo = &fl->redo;
    hipError_t e = hipSuccess;
    auto pass = [&](bool strict, int64_t blocks, int64_t every) -> mxl_status {
        hf = {INT_MAX, 0, 0, 0, 0};
        if ((e = hipMemcpyAsync(fl, &hf, sizeof hf, hipMemcpyHostToDevice, s)) != hipSuccess ||
            (e = bj_invert(*A, bs, adaptive ? 1 : 0, accuracy, (double *)J->bcond->p, prec, &fl->bad, out, strict,
                           blocks, every, s)) != hipSuccess)
            return set_error(MXL_ERR_DEVICE, std::string("block inversion: ") + hipGetErrorString(e));
        if (out.store) hipLaunchKernelGGL(k_bj_offsets, dim3((unsigned)((nb + 255) / 256)), dim3(256), 0, s, nb,
                                          out.stride, off);
        if (out.inv) {  // offsets of mixed precisions, read back with the flags
            const int g = (int)std::min<int64_t>(kScanGrid, (nb + kScanWG - 1) / kScanWG);
            const int64_t chunk = (nb + g - 1) / g;
            if (g > 1) hipLaunchKernelGGL(k_bj_sizes, dim3(g), dim3(kScanWG), 0, s, nb, chunk, bs, prec, sums);
            hipLaunchKernelGGL(k_bj_scan, dim3(g), dim3(kScanWG), 0, s, nb, chunk, bs, prec, sums, off, &fl->total);
        }
        if ((e = hipGetLastError()) != hipSuccess ||
            (e = hipMemcpyAsync(&hf, fl, sizeof hf, hipMemcpyDeviceToHost, s)) != hipSuccess ||
            (e = hipStreamSynchronize(s)) != hipSuccess)
            return set_error(MXL_ERR_DEVICE, std::string("block inversion read-back: ") + hipGetErrorString(e));
        return MXL_OK;
    };
    constexpr int64_t kLook = 1024;
    mxl_status st = MXL_OK;
    BufPtr tmp;
    bool mixed = false;
    if (adaptive && nb > 4 * kLook && nb * out.stride >= (int64_t)16 << 20) {
        if ((st = pass(false, kLook, nb / kLook)) != MXL_OK) return st;
        mixed = hf.mixed != 0;
    } else if (adaptive) {
        mixed = true;  // small: the copy costs less than a guess that fails
    }
    for (bool strict = false;;) {
        if (mixed && !tmp) {
            J->bstore.reset();
            out.store = nullptr;
            if (!(tmp = mk(nb * bs * bs * 8))) return set_error(MXL_ERR_OUT_OF_MEMORY, "block Jacobi workspace");
            out.inv = (double *)tmp->p;
        } else if (!mixed && !J->bstore) {
            J->bstore_bytes = nb * out.stride;
            if (!(J->bstore = mk(J->bstore_bytes))) return set_error(MXL_ERR_OUT_OF_MEMORY, "block Jacobi storage");
            out.store = (unsigned char *)J->bstore->p;
        }
        if ((st = pass(strict, nb, 1)) != MXL_OK) return st;
        if (hf.redo && !strict) strict = true;
        else if (hf.mixed && !mixed) mixed = true;
        else break;
    }
    if (hf.bad != INT_MAX) {
        char msg[96];
        snprintf(msg, sizeof msg, "diagonal block %d is singular", hf.bad);
        return set_error(MXL_ERR_ZERO_DIAG, msg);
    }
    if (tmp) {
        if (!(J->bstore = mk(hf.total))) return set_error(MXL_ERR_OUT_OF_MEMORY, "block Jacobi storage");
        J->bstore_bytes = hf.total;
        if ((e = bj_pack(bs, nb, (const double *)tmp->p, prec, off, (unsigned char *)J->bstore->p, s)) != hipSuccess ||
            (e = hipStreamSynchronize(s)) != hipSuccess)
            return set_error(MXL_ERR_DEVICE, std::string("block Jacobi packing: ") + hipGetErrorString(e));
    }
    auto *op = new mxl_op;
    op->kind = MXL_OP_JACOBI;
    op->jac = J;
    *Pout = op;
    return MXL_OK;
} catch (...) {
    return mxl::abi_exception(__func__);
}

namespace {

BufPtr dev_buf(size_t bytes) {
    auto d = std::make_shared<DevBuf>();
    if (hipMalloc(&d->p, bytes ? bytes : 16) != hipSuccess) return BufPtr();
    d->bytes = bytes;
    d->owned = true;
    return d;
}

// Supervariable agglomeration: runs of rows with one column set (same[i]:
// row i continues the run of row i - 1), each cut into pieces of at most
// max_bs rows, packed in row order into blocks of at most max_bs rows (a
// piece that does not fit starts the next block).
std::vector<int32_t> agglomerate(const std::vector<unsigned char> &same, int max_bs) {
    const int64_t n = (int64_t)same.size();
    std::vector<int32_t> bp{0};
    int64_t fill = 0;
    for (int64_t i = 0; i < n;) {
        int64_t e = i + 1;
        while (e < n && same[(size_t)e]) ++e;
        for (int64_t p = i; p < e; p += max_bs) {
            const int64_t len = std::min<int64_t>(max_bs, e - p);
            if (fill > 0 && fill + len > max_bs) {
                bp.push_back((int32_t)p);
                fill = 0;
            }
            fill += len;
        }
        i = e;
    }
    bp.push_back((int32_t)n);
    return bp;
}

// Generation over given boundaries (block sizes 1..32): per size class a
// list of its blocks and one launch of the class's elimination kernel, then
// the precision read-back, the 16-byte-aligned offsets and the packing.
mxl_status bj_generate_var(const std::shared_ptr<MatrixImpl> &A, std::vector<int32_t> bp, int adaptive,
                           double accuracy, mxl_op **Pout) {
    hipStream_t s = A->ctx->stream;
    const int64_t nb = (int64_t)bp.size() - 1;
    static const int kClass[6] = {1, 2, 4, 8, 16, 32};
    std::vector<int> list;
    list.reserve((size_t)nb);
    int64_t cstart[7] = {0};
    std::vector<int64_t> toff((size_t)nb + 1, 0);
    for (int64_t b = 0; b < nb; ++b) {
        const int64_t m = bp[(size_t)b + 1] - bp[(size_t)b];
        toff[(size_t)b + 1] = toff[(size_t)b] + m * m;
    }
    for (int c = 0; c < 6; ++c) {
        cstart[c] = (int64_t)list.size();
        const int lo = c == 0 ? 1 : kClass[c - 1] + 1, hi = kClass[c];
        for (int64_t b = 0; b < nb; ++b) {
            const int m = bp[(size_t)b + 1] - bp[(size_t)b];
            if (m >= lo && m <= hi) list.push_back((int)b);
        }
    }
    cstart[6] = (int64_t)list.size();
    auto J = std::make_shared<JacobiImpl>();
    J->A = A;
    J->block = true;
    J->var = true;
    J->bs = 0;
    J->nblocks = nb;
    BufPtr dlist = dev_buf(list.size() * 4), dtoff = dev_buf((size_t)(nb + 1) * 8),
           tmp = dev_buf((size_t)toff[(size_t)nb] * 8), flags = dev_buf(8);
    J->bptr_d = dev_buf((size_t)(nb + 1) * 4);
    J->rblk = dev_buf((size_t)A->nrows * 4);
    J->bcond = dev_buf((size_t)nb * 8);
    J->bprec = dev_buf((size_t)nb * 4);
    J->boff = dev_buf((size_t)nb * 8);
    if (!dlist || !dtoff || !tmp || !flags || !J->bptr_d || !J->rblk || !J->bcond || !J->bprec || !J->boff)
        return set_error(MXL_ERR_OUT_OF_MEMORY, "block Jacobi workspace");
    hipError_t e;
    if ((e = hipMemcpyAsync(dlist->p, list.data(), list.size() * 4, hipMemcpyHostToDevice, s)) != hipSuccess ||
        (e = hipMemcpyAsync(dtoff->p, toff.data(), (size_t)(nb + 1) * 8, hipMemcpyHostToDevice, s)) != hipSuccess ||
        (e = hipMemcpyAsync(J->bptr_d->p, bp.data(), (size_t)(nb + 1) * 4, hipMemcpyHostToDevice, s)) !=
            hipSuccess)
        return set_error(MXL_ERR_DEVICE, std::string("block Jacobi upload: ") + hipGetErrorString(e));
    const int *rp = (const int *)A->row_ptr->p, *col = (const int *)A->col->p;
    const double *val = (const double *)A->val->p;
    double *cond = (double *)J->bcond->p;
    int *prec = (int *)J->bprec->p, *fl = (int *)flags->p;
    BlockOut out{};
    out.inv = (double *)tmp->p;
    out.redo = fl + 1;
    int hf[2];  // lowest singular block, whether to invert strictly
    std::vector<int> hp((size_t)nb);
    for (int strict = 0; strict < 2; ++strict) {
        hf[0] = INT_MAX;
        hf[1] = 0;
        if ((e = hipMemcpyAsync(fl, hf, 8, hipMemcpyHostToDevice, s)) != hipSuccess)
            return set_error(MXL_ERR_DEVICE, std::string("block Jacobi upload: ") + hipGetErrorString(e));
        for (int c = 0; c < 6; ++c) {
            const int64_t cnt = cstart[c + 1] - cstart[c];
            if (cnt == 0) continue;
            const BlockSel sel{(const int *)dlist->p + cstart[c], (const int *)J->bptr_d->p,
                               (const int64_t *)dtoff->p, 1};
            const int per = kWave / (kClass[c] < 16 ? kClass[c] : 16);  // blocks of a wave
            const dim3 g((unsigned)((cnt + per - 1) / per));
            auto run = [&]() -> hipError_t {
                if (strict) {
                    MXL_BS_SWITCH(kClass[c], hipLaunchKernelGGL((k_bj_invert<BS, true, true>), g, dim3(kWave), 0, s,
                                                                A->nrows, rp, col, val, adaptive, accuracy, cond, prec,
                                                                fl, sel, cnt, out));
                } else {
                    MXL_BS_SWITCH(kClass[c], hipLaunchKernelGGL((k_bj_invert<BS, true, false>), g, dim3(kWave), 0, s,
                                                                A->nrows, rp, col, val, adaptive, accuracy, cond, prec,
                                                                fl, sel, cnt, out));
                }
                return hipGetLastError();
            };
            if ((e = run()) != hipSuccess)
                return set_error(MXL_ERR_DEVICE, std::string("block inversion: ") + hipGetErrorString(e));
        }
        if (!strict)
            hipLaunchKernelGGL(k_bj_rowmap, dim3((unsigned)((nb + 255) / 256)), dim3(256), 0, s, nb,
                               (const int *)J->bptr_d->p, (int *)J->rblk->p);
        if ((e = hipGetLastError()) != hipSuccess ||
            hipMemcpyAsync(hf, fl, 8, hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipMemcpyAsync(hp.data(), J->bprec->p, (size_t)nb * 4, hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess)
            return set_error(MXL_ERR_DEVICE, "block inversion read-back");
        if (!hf[1]) break;
    }
    const int hb = hf[0];
    if (hb != INT_MAX) {
        char msg[96];
        snprintf(msg, sizeof msg, "diagonal block %d is singular", hb);
        return set_error(MXL_ERR_ZERO_DIAG, msg);
    }
    std::vector<int64_t> ho((size_t)nb);
    int64_t total = 0;
    for (int64_t b = 0; b < nb; ++b) {
        const int m = bp[(size_t)b + 1] - bp[(size_t)b];
        ho[(size_t)b] = total;
        total += (int64_t)m * bjv_chunks(m, hp[(size_t)b]) * 16;
    }
    J->bstore = dev_buf((size_t)total);
    if (!J->bstore) return set_error(MXL_ERR_OUT_OF_MEMORY, "block Jacobi storage");
    J->bstore_bytes = total;
    if ((e = hipMemcpyAsync(J->boff->p, ho.data(), (size_t)nb * 8, hipMemcpyHostToDevice, s)) != hipSuccess)
        return set_error(MXL_ERR_DEVICE, "block Jacobi offsets");
    hipLaunchKernelGGL(k_bj_pack_var, dim3((unsigned)nb), dim3(kWave), 0, s, nb, (const int *)J->bptr_d->p,
                       (const int64_t *)dtoff->p, (const double *)tmp->p, (const int *)J->bprec->p,
                       (const int64_t *)J->boff->p, (unsigned char *)J->bstore->p);
    if ((e = hipGetLastError()) != hipSuccess || (e = hipStreamSynchronize(s)) != hipSuccess)
        return set_error(MXL_ERR_DEVICE, std::string("block Jacobi packing: ") + hipGetErrorString(e));
    J->bptr_h = std::move(bp);
    auto *op = new mxl_op;
    op->kind = MXL_OP_JACOBI;
    op->jac = J;
    *Pout = op;
    return MXL_OK;
}

}  // namespace

extern "C" mxl_status mxl_bjacobi_generate_var(const mxl_op *Aop, int64_t nblocks, const int32_t *bptr_host,
                                               int32_t max_block_size, int32_t adaptive, double accuracy,
                                               mxl_op **Pout) try {
    if (!Aop || !Pout || Aop->kind != MXL_OP_MATRIX)
        return set_error(MXL_ERR_INVALID_ARG, "matrix operator and output required");
    *Pout = nullptr;
    const auto &A = Aop->mat;
    if (A->nrows != A->ncols) return set_error(MXL_ERR_NOT_IMPLEMENTED, "block Jacobi needs a square matrix");
    if (A->dtype != MXL_F64) return set_error(MXL_ERR_NOT_IMPLEMENTED, "block Jacobi needs an FP64 matrix");
    if (A->format == MXL_FMT_STENCIL)
        return set_error(MXL_ERR_NOT_IMPLEMENTED, "block Jacobi needs stored matrix rows");
    if (A->nrows == 0) return set_error(MXL_ERR_INVALID_ARG, "empty matrix");
    if (!(accuracy >= 0.0)) return set_error(MXL_ERR_INVALID_ARG, "accuracy must be >= 0");
    if (accuracy == 0.0) accuracy = 0.1;
    const int64_t n = A->nrows;
    DeviceScope ds(A->ctx->device);
    hipStream_t s = A->ctx->stream;
    std::vector<int32_t> bp;
    if (bptr_host) {
        if (nblocks < 1 || nblocks > n) return set_error(MXL_ERR_INVALID_ARG, "1 <= nblocks <= nrows required");
        bp.assign(bptr_host, bptr_host + nblocks + 1);
        if (bp[0] != 0 || bp[(size_t)nblocks] != n)
            return set_error(MXL_ERR_INVALID_ARG, "block boundaries must run from 0 to nrows");
        for (int64_t b = 0; b < nblocks; ++b) {
            const int64_t m = (int64_t)bp[(size_t)b + 1] - bp[(size_t)b];
            if (m < 1 || m > kBjMax) {
                char msg[112];
                snprintf(msg, sizeof msg, "block %lld has %lld rows (1 to %d allowed)", (long long)b,
                         (long long)m, kBjMax);
                return set_error(MXL_ERR_INVALID_ARG, msg);
            }
        }
    } else {
        if (max_block_size < 1 || max_block_size > kBjMax)
            return set_error(MXL_ERR_INVALID_ARG, "max_block_size must be 1..32");
        BufPtr same = dev_buf((size_t)n);
        if (!same) return set_error(MXL_ERR_OUT_OF_MEMORY, "supervariable flags");
        hipLaunchKernelGGL(k_bj_same_prev, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n,
                           (const int *)A->row_ptr->p, (const int *)A->col->p, (unsigned char *)same->p);
        std::vector<unsigned char> h((size_t)n);
        if (hipGetLastError() != hipSuccess ||
            hipMemcpyAsync(h.data(), same->p, (size_t)n, hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess)
            return set_error(MXL_ERR_DEVICE, "supervariable detection");
        bp = agglomerate(h, max_block_size);
    }
    return bj_generate_var(A, std::move(bp), adaptive ? 1 : 0, accuracy, Pout);
} catch (...) {
    return mxl::abi_exception(__func__);
}

extern "C" mxl_status mxl_bjacobi_blocks(const mxl_op *Pop, int32_t *bptr_host) try {
    if (!Pop || Pop->kind != MXL_OP_JACOBI || !Pop->jac->block || !bptr_host)
        return set_error(MXL_ERR_INVALID_ARG, "block-Jacobi operator and output required");
    const JacobiImpl &J = *Pop->jac;
    if (J.var) {
        std::copy(J.bptr_h.begin(), J.bptr_h.end(), bptr_host);
    } else {
        for (int64_t b = 0; b <= J.nblocks; ++b) bptr_host[b] = (int32_t)std::min<int64_t>(b * J.bs, J.A->nrows);
    }
    return MXL_OK;
} catch (...) {
    return mxl::abi_exception(__func__);
}

extern "C" mxl_status mxl_bjacobi_info(const mxl_op *Pop, int64_t *nblocks, double *cond_host,
                                       int32_t *precision_host, double *inv_host, int64_t *storage_bytes) try {
    if (!Pop || Pop->kind != MXL_OP_JACOBI || !Pop->jac->block)
        return set_error(MXL_ERR_INVALID_ARG, "not a block-Jacobi operator");
    const JacobiImpl &J = *Pop->jac;
    DeviceScope ds(J.A->ctx->device);
    hipStream_t s = J.A->ctx->stream;
    const int64_t nb = J.nblocks, bs = J.bs, n = J.A->nrows;
    if (nblocks) *nblocks = nb;
    if (storage_bytes) *storage_bytes = J.bstore_bytes;
    if (cond_host && hipMemcpyAsync(cond_host, J.bcond->p, (size_t)nb * 8, hipMemcpyDeviceToHost, s) != hipSuccess)
        return set_error(MXL_ERR_DEVICE, "copy condition numbers");
    std::vector<int> hp((size_t)nb);
    if (hipMemcpyAsync(hp.data(), J.bprec->p, (size_t)nb * 4, hipMemcpyDeviceToHost, s) != hipSuccess)
        return set_error(MXL_ERR_DEVICE, "copy precisions");
    std::vector<unsigned char> store;
    std::vector<int64_t> ho;
    if (inv_host) {
        store.resize((size_t)J.bstore_bytes);
        ho.resize((size_t)nb);
        if (hipMemcpyAsync(store.data(), J.bstore->p, store.size(), hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipMemcpyAsync(ho.data(), J.boff->p, (size_t)nb * 8, hipMemcpyDeviceToHost, s) != hipSuccess)
            return set_error(MXL_ERR_DEVICE, "copy inverses");
    }
    if (hipStreamSynchronize(s) != hipSuccess) return set_error(MXL_ERR_DEVICE, "block Jacobi read-back");
    if (precision_host)
        for (int64_t b = 0; b < nb; ++b) precision_host[b] = hp[b];
    if (inv_host) {  // packed m x m per block, as FP64
        int64_t o = 0;
        for (int64_t b = 0; b < nb; ++b) {
            const int64_t m = J.var ? J.bptr_h[(size_t)b + 1] - J.bptr_h[(size_t)b] : std::min(bs, n - b * bs);
            // elements per stored row: bs (uniform) or whole 16-byte chunks (variable)
            const int64_t ld = J.var ? (int64_t)bjv_chunks((int)m, hp[b]) * (hp[b] == BJ_P16 ? 8 : hp[b] == BJ_P32 ? 4 : 2)
                                     : bs;
            const unsigned char *base = store.data() + ho[b];
            for (int64_t i = 0; i < m; ++i)
                for (int64_t jj = 0; jj < m; ++jj) {
                    const int64_t k = i * ld + jj;
                    double x;
                    if (hp[b] == BJ_P16) {
                        _Float16 h;
                        std::memcpy(&h, base + 2 * k, 2);
                        x = (double)h;
                    } else if (hp[b] == BJ_P32) {
                        float f;
                        std::memcpy(&f, base + 4 * k, 4);
                        x = f;
                    } else {
                        std::memcpy(&x, base + 8 * k, 8);
                    }
                    inv_host[o++] = x;
                }
        }
    }
    return MXL_OK;
} catch (...) {
    return mxl::abi_exception(__func__);
}
