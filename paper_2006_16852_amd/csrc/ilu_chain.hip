// ilu_chain.hip -- exact triangular solves of the ILU-type preconditioner
// (Sec. 3.2) for factors whose rows form chains, in one launch per triangle
// without levels.
//
// A chain is a maximal run of consecutive rows each of which depends on its
// neighbour (the row before it in L, the row after it in U); on a grid
// numbered line by line a chain is a grid line.  The substitution inside a
// chain is sequential whatever the schedule, so one lane solves one chain and
// its latest value never leaves a register; all other operands come from
// lanes that run beside it.  A workgroup owns a group of at most 64 chains:
//
//  * One worker wave, lane = chain.  A pass over the wave solves the next row
//    of every chain whose operands are there.  It touches LDS only: solved
//    values of the group's own rows, and records that the loaders prepare.
//  * Loader waves, NL / C lanes per chain, each lane one row ahead of the
//    other.  A lane loads its row's entries, polls the operands that other
//    groups produce until they arrive, and writes the row's record: right-hand
//    side, coefficient of the chain neighbour, and for every other entry a
//    coefficient and an LDS operand (for an operand of another group the
//    finished product, with the constant 1 as operand).
//
// What bounds it is the dependency chain, not bytes: 382 rows after another
// on a 128^3 grid (0.27 us each, the worker's pass: two LDS round trips and
// some 75 instructions) plus the hops from group to group through memory
// (2 us each: store, poll, record).  Groups are therefore two-dimensional
// tiles of chains where the numbering allows (8 x 8 grid lines: 30 hops
// instead of 128).  128^3 convection-diffusion, both triangles: 485 us, of
// which the level-scheduled launches took 2,740 us (4.3 us per level); with
// 64 consecutive chains per group 1,050 us.  700^2 5-point: 1,040 us against
// 5,560 us.
//
// Values of other groups are their own flags: y and z are filled with a NaN
// pattern that no result carries (a result with that pattern is replaced by
// an ordinary NaN), stored with device-scope atomics as they are solved, and
// polled until the pattern is gone.
//
// No wait can be circular: groups take tickets in solve order, every operand
// of a group lies in the group itself or in one with an earlier ticket
// (checked at generation for the tiled order), a ticket is held by a
// workgroup that runs, and no lane waits inside a branch for another lane of
// its wave (every pass tries once and goes on).  As a backstop a workgroup
// whose worker solves no row for trs_wait_passes(n) passes gives up: it turns
// its unsolved rows into NaN, sets the flag behind the tickets and ends.  The
// worker alone counts (the loaders end with it), and its limit grows with n: a
// group may have to wait until all rows before it are solved one after another.
// The flag is an error of the next call that synchronises (mxl_ilu_info and
// GMRES solves).
#include <algorithm>
#include <climits>
#include <string>
#include <vector>

#include "device_common.hpp"
#include "internal.hpp"

namespace mxl {

constexpr unsigned kTrsWaitHi = 0x7ff4a5a5u;  // a signalling NaN: no arithmetic yields it
constexpr unsigned long long kTrsWaitBits = 0x7ff4a5a55a5a5a5aull;
constexpr int kTrsPad = 0x7fffffff;           // code of an empty slot
constexpr int kTrsLanes = 64;                 // worker lanes = chains of a group
constexpr int kTrsTJ = 8;                     // tile of chains along the numbering
constexpr size_t kTrsLdsMax = 158 * 1024;

// Record shapes: entries besides the chain neighbour, loader lanes, ring
// depth in rows per loader lane.  The narrow shape serves 5- and 7-point
// patterns, the wide one up to the 12 of a 27-point one.
constexpr int kTrsNarrow = 3, kTrsWide = 12;
constexpr int kTrsLoaders = 256;

// Passes of a worker without progress before it gives up.  A pass takes at least
// 0.15 us and a row, solved alone, at most some 3 us (a hop through memory), so
// 64 passes a row cannot run out before all n rows are solved.
constexpr int64_t trs_wait_passes(int64_t n) { return ((int64_t)1 << 26) + 64 * n; }

__device__ __forceinline__ bool trs_ready(double v) { return (unsigned)__double2hiint(v) != kTrsWaitHi; }
__device__ __forceinline__ double trs_wait() { return __longlong_as_double((long long)kTrsWaitBits); }
__device__ __forceinline__ double trs_pub(double v) { return trs_ready(v) ? v : (double)__builtin_nan(""); }
template <typename T>
__device__ __forceinline__ T lds_get(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
template <typename T>
__device__ __forceinline__ void lds_put(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// The order of relaxed LDS accesses around a flag: no instructions, as LDS serves
// a wave's accesses in the order in which they are issued.
__device__ __forceinline__ void order_after() { __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront"); }
__device__ __forceinline__ void order_before() { __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront"); }
__device__ __forceinline__ double mem_get(const double *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void mem_put(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One triangle as the kernel reads it.  Entries besides the diagonal and the
// chain neighbour are slot-major in column order, slot s of row i at
// s * n_pad + i; code: an operand's column (>= 0: produced by another group,
// or beyond the group's LDS places), 0x80000000 | its LDS place, or kTrsPad.
struct TrsView {
    int64_t n_pad;
    const int *code;
    const double *val, *prev, *diag;
    int w;
    const int *cstart;       // chain t holds rows cstart[t] .. cstart[t + 1] - 1
    const int *cbase;        // LDS place of its first solved row
    const int *glist, *gptr; // group g: chains glist[gptr[g]] .. glist[gptr[g + 1] - 1]
    int groups, C, cap;
    int fail;                // place of the give-up flag after this triangle's ticket
    int64_t passes;          // a worker's passes without progress before it gives up
};

template <bool LOWER, int NE, int NL, int RD>
constexpr size_t trs_lds_bytes(int cap) {
    return (size_t)(cap + 1) * 8 + (size_t)NL * RD * (8 + 8 + (LOWER ? 0 : 8) + 12 * NE);
}

// LOWER: x = L^{-1} b, rows ascending, and znext is filled with the wait
// pattern for the upper solve.  Otherwise x = U^{-1} b, rows descending, and
// out = alpha x + beta out.  The arithmetic of a row is the sequential one in
// column order without contraction.
template <bool LOWER, int NE, int NL, int RD>
__global__ __launch_bounds__(kTrsLanes + NL) void k_trs_chain(TrsView M, const double *__restrict__ b, double *x,
                                                              double *__restrict__ znext, double alpha, double beta,
                                                              double *__restrict__ out, unsigned *ticket) {
#pragma clang fp contract(off)
    extern __shared__ double lds[];
    __shared__ int s_tk, s_abort;
    constexpr int NS = NL * RD;  // records
    const int cap = M.cap, C = M.C, one = cap;
    // solved values (cap places and the constant 1), then the records
    double *xl = lds, *rs = xl + cap + 1, *rvp = rs + NS, *rv = rvp + NS, *rd = rv + NE * NS;
    int *rl = (int *)(rd + (LOWER ? 0 : NS));
    const int tid = threadIdx.x;
    if (tid == 0) {
        s_tk = (int)atomicAdd(ticket, 1u);
        s_abort = 0;
    }
    for (int j = tid; j < cap + 1 + NS; j += kTrsLanes + NL) lds[j] = j == one ? 1.0 : trs_wait();
    __syncthreads();
    if (s_tk >= M.groups) return;
    const int g = LOWER ? s_tk : M.groups - 1 - s_tk;
    const int q0 = M.gptr[g], nc = M.gptr[g + 1] - q0;
    const int D = NL / C, RB = D * RD;  // loader lanes and ring slots per chain
    if (tid >= kTrsLanes) {  // ---------------------------------------- loaders
        const int lid = tid - kTrsLanes, ch = lid / D, o = lid % D;
        const bool on = ch < nc;
        const int t = on ? M.glist[q0 + ch] : 0;
        const int cs = on ? M.cstart[t] : 0, len = on ? M.cstart[t + 1] - cs : 0;
        int c[NE], cn[NE];  // the row in hand and, already under way, the lane's next one
        double v[NE], vn[NE], xr[NE];
        double s = 0.0, sn = 0.0, d = 1.0, dn = 1.0, vp = 0.0, vpn = 0.0;
        unsigned need = 0;  // operands not yet seen
        int p = o;
        auto fetch = [&](int pp) {
            if (pp < len) {
                const int i = LOWER ? cs + pp : cs + len - 1 - pp;
#pragma unroll
                for (int m = 0; m < NE; ++m) {
                    cn[m] = m < M.w ? M.code[(int64_t)m * M.n_pad + i] : kTrsPad;
                    vn[m] = m < M.w ? M.val[(int64_t)m * M.n_pad + i] : 0.0;
                }
                vpn = M.prev[i];
                sn = b[i];
                if (!LOWER) dn = M.diag[i];
            }
        };
        auto take = [&]() {
            need = 0;
#pragma unroll
            for (int m = 0; m < NE; ++m) {
                c[m] = cn[m];
                v[m] = vn[m];
                if (c[m] >= 0 && c[m] != kTrsPad) need |= 1u << m;
                xr[m] = 1.0;
            }
            s = sn;
            d = dn;
            vp = vpn;
        };
        bool act = p < len;
        fetch(p);
        if (act) take();
        fetch(p + D);
        while (__any(act)) {
            double xp[NE];
#pragma unroll
            for (int m = 0; m < NE; ++m) xp[m] = act && (need >> m & 1) ? mem_get(x + c[m]) : trs_wait();
            // ring slots row by row over the chains: the worker's lanes read neighbouring ones
            const int idx = act ? (p & (RB - 1)) * C + ch : 0;
            const bool empty = act && !trs_ready(lds_get(rs + idx));
#pragma unroll
            for (int m = 0; m < NE; ++m)
                if (trs_ready(xp[m])) {
                    xr[m] = xp[m];
                    need &= ~(1u << m);
                }
            const bool pub = act && need == 0 && empty;
            if (pub) {
#pragma unroll
                for (int m = 0; m < NE; ++m) {
                    const bool pad = c[m] == kTrsPad, loc = c[m] < 0;
                    lds_put(rl + m * NS + idx, loc ? c[m] & kTrsPad : one);
                    lds_put(rv + m * NS + idx, pad ? 0.0 : loc ? v[m] : v[m] * xr[m]);
                }
                lds_put(rvp + idx, vp);
                if (!LOWER) lds_put(rd + idx, d);
                // the right-hand side is the record's flag: written last
                __hip_atomic_store(rs + idx, trs_pub(s), __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
                p += D;
                act = p < len;
                if (act) take();
                fetch(p + D);
            }
            if (!__any(pub) && lds_get(&s_abort)) break;  // the worker has given up
        }
        return;
    }
    // ------------------------------------------------------------- the worker
    __builtin_amdgcn_s_setprio(3);  // its passes are the critical path
    const bool on = tid < nc;
    const int t = on ? M.glist[q0 + tid] : 0;
    const int cs = on ? M.cstart[t] : 0, len = on ? M.cstart[t + 1] - cs : 0;
    int pl = on ? M.cbase[t] : 0;
    int p = 0, seen = 0;
    int64_t idle = 0;  // passes since a row was solved, counted beside the passes that solve one
    int i = LOWER ? cs : cs + len - 1;
    int idx = on ? tid : 0;
    double yprev = 0.0;
    bool act = p < len;
    // the loads above are done: without this the loop waits for all its own
    // stores in every pass (vmcnt 0, the other counters untouched)
    __builtin_amdgcn_s_waitcnt(0xF70);
    while (__any(act)) {
        bool ok;
        do {
            // the flag first: LDS serves a wave in order, so a record read after
            // a set flag is whole; the fence holds the compiler to that order
            double s = lds_get(rs + idx);
            order_after();
            int l[NE];
            double xv[NE], vv[NE];
#pragma unroll
            for (int m = 0; m < NE; ++m) l[m] = lds_get(rl + m * NS + idx);
#pragma unroll
            for (int m = 0; m < NE; ++m) vv[m] = lds_get(rv + m * NS + idx);
            const double vp = lds_get(rvp + idx);
            double dd = 1.0;
            if (!LOWER) dd = lds_get(rd + idx);
            ok = act && trs_ready(s);
#pragma unroll
            for (int m = 0; m < NE; ++m) xv[m] = lds_get(xl + (ok ? l[m] : one));
#pragma unroll
            for (int m = 0; m < NE; ++m) ok = ok && trs_ready(xv[m]);
            // column order: the neighbour is the last entry of L, the first of U;
            // a chain's first row has none (coefficient and yprev are 0)
            if (!LOWER) s = s - vp * yprev;
#pragma unroll
            for (int m = 0; m < NE; ++m) s = s - vv[m] * xv[m];
            if (LOWER) s = s - vp * yprev;
            if (ok) {
                if (!LOWER) s = s / dd;
                yprev = trs_pub(s);
                if (pl < cap) lds_put(xl + pl, yprev);
                mem_put(x + i, yprev);
                order_before();                 // the record has been read
                lds_put(rs + idx, trs_wait());  // the slot is free again
                if (LOWER) {
                    znext[i] = trs_wait();
                } else if (beta == 0.0) {
                    out[i] = alpha * yprev;
                } else {
                    out[i] = alpha * yprev + beta * out[i];
                }
                ++p;
                ++pl;
                i += LOWER ? 1 : -1;
                act = p < len;
                idx = act ? (idx + C) & (NS - 1) : 0;  // the next ring slot: NS = RB * C
            }
        } while (__any(ok));
        if (__any(p != seen)) {
            seen = p;
            idle = 0;
        } else if (++idle > M.passes) {
            lds_put(&s_abort, 1);
            if (tid == 0) mem_put((int *)ticket + M.fail, 1);
            break;
        }
    }
    for (; p < len; ++p, i += LOWER ? 1 : -1) {  // the backstop: also ends the waits of later groups
        mem_put(x + i, (double)__builtin_nan(""));
        if (LOWER) znext[i] = trs_wait();
        else out[i] = (double)__builtin_nan("");
    }
}

// tickets: one of each triangle, then the give-up flag
__global__ void k_trs_begin(int64_t n, double *__restrict__ y, unsigned *tickets) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < 2) tickets[i] = 0;
    if (i < n) y[i] = trs_wait();
}

__global__ void k_trs_clear(unsigned *tickets) {
    if (threadIdx.x < 3) tickets[threadIdx.x] = 0;
}

// ------------------------------------------------------------ generation
// What the plan of one triangle is made from, gathered on the device.
struct TrsInfo {
    int w;       // widest row (entries besides the diagonal and the chain neighbour)
    int lo, hi;  // smallest and largest distance, in chains, of an operand more than one chain away
    int longest; // rows of the longest chain
    int nch;     // chains
    int bad;     // 1: two-dimensional tiles would not be in solve order
    int faults;  // kTrsUnsorted, kTrsOutside: what the column indices violate
};
constexpr int kTrsUnsorted = 1, kTrsOutside = 2;

// The groups of a triangle: `groups` runs of C consecutive chains, or (W > 0)
// tiles of kTrsTJ x TK chains of the chains laid out as (t % W, t / W), the
// columns shifted by skew per row, tile rows of NJ tiles.
struct TrsPlan {
    int ok, wide, places, C, W, skew, TK, NJ, groups;
};

__host__ __device__ inline void trs_count_groups(TrsPlan &p, int nch) {
    if (p.W == 0) {
        p.NJ = 0;
        p.groups = (nch + p.C - 1) / p.C;
        return;
    }
    const int K = (nch - 1) / p.W;
    p.NJ = (p.W - 1 + p.skew * K) / kTrsTJ + 1;
    p.groups = p.NJ * (K / p.TK + 1);
}

__host__ __device__ inline TrsPlan trs_plan(int64_t n, const TrsInfo &f) {
    TrsPlan p{};
    // Chains shorter than 8 rows on average keep the worker's lanes waiting
    // for records, and rows wider than a record do not fit it: such factors
    // (random patterns, node blocks) have few levels, which the level
    // launches serve.
    // Rows out of order have no place here: an entry on the wrong side of the
    // diagonal would be waited for in a circle, and one next to the diagonal's
    // place would be taken for the chain neighbour.
    p.ok = !f.faults && f.nch >= 1 && n / f.nch >= 8 && f.w <= kTrsWide;
    if (!p.ok) return p;
    p.wide = f.w > kTrsNarrow;
    const size_t rec = p.wide ? trs_lds_bytes<false, kTrsWide, kTrsLoaders, 1>(0)
                              : trs_lds_bytes<false, kTrsNarrow, kTrsLoaders, 2>(0);
    p.places = (int)((kTrsLdsMax - rec) / 8) - 1;
    // As many chains per group as its LDS holds (fewer hops between groups):
    // 64 of 128 rows take 64 KB.
    p.C = kTrsLanes;
    while (p.C > 4 && (int64_t)p.C * (n / f.nch) > p.places - p.places / 8) p.C /= 2;
    p.TK = p.C / kTrsTJ;
    if (p.TK > 1 && f.hi > 0) {  // operands further than one chain away: a plane of chains lies between
        const int mid = (int)(((int64_t)f.lo + f.hi) / 2), sk = mid - f.lo;
        if (mid >= kTrsTJ && mid < f.nch && sk <= 4 && (int64_t)f.nch / mid * sk <= 8 * (int64_t)mid) {
            p.W = mid;
            p.skew = sk;
        }
    }
    trs_count_groups(p, f.nch);
    return p;
}

// Chains of group g, ascending.
template <typename F>
__device__ __forceinline__ void trs_group(const TrsPlan &p, int nch, int g, F f) {
    if (p.W == 0) {
        for (int t = g * p.C; t < nch && t < (g + 1) * p.C; ++t) f(t);
        return;
    }
    const int J = g % p.NJ, K = g / p.NJ;
    for (int k = K * p.TK; k < (K + 1) * p.TK; ++k)
        for (int e = 0; e < kTrsTJ; ++e) {
            const int64_t j = (int64_t)J * kTrsTJ + e - (int64_t)p.skew * k, t = (int64_t)k * p.W + j;
            if (j >= 0 && j < p.W && t < nch) f((int)t);
        }
}

// What a generation reads back at once, in the order of the copy.
struct TrsHead {
    int bad;       // first row with a missing or zero diagonal
    int widths[2];
    TrsInfo f[2];  // of L and of U
};

__global__ void k_ilu_begin(TrsHead *h) {
    if (threadIdx.x == 0) {
        h->bad = INT_MAX;
        h->widths[0] = h->widths[1] = 0;
    }
    if (threadIdx.x < 2) h->f[threadIdx.x] = TrsInfo{0, INT_MAX, 0, 0, 0, 0, 0};
}

// Both triangles in every launch (blockIdx.y: 0 the lower, 1 the upper): the plan
// of a small system costs its launches.
struct TrsPair {
    int *sums[2], *rowchain[2], *cstart[2];
};

// Row i opens a chain: in L when it has no entry i - 1, in U when row i - 1
// has no entry i (chains are listed by ascending rows in both).
__device__ __forceinline__ bool trs_head(bool lower, int64_t i, const int *__restrict__ rp,
                                         const int *__restrict__ col, const int *__restrict__ dpos) {
    if (i == 0) return true;
    if (lower) return !(dpos[i] > rp[i] && col[dpos[i] - 1] == (int)i - 1);
    return !(dpos[i - 1] + 1 < rp[i] && col[dpos[i - 1] + 1] == (int)i);
}

constexpr int kTrsScan = 1024;  // rows per workgroup of the two scan passes

__global__ __launch_bounds__(kWG) void k_trs_count(int64_t n, const int *__restrict__ rp,
                                                   const int *__restrict__ col, const int *__restrict__ dpos,
                                                   TrsPair q) {
    __shared__ int part[kWG / kWave];
    const bool lower = blockIdx.y == 0;
    int *sums = q.sums[blockIdx.y];
    int h = 0;
    for (int e = 0; e < kTrsScan / kWG; ++e) {
        const int64_t i = (int64_t)blockIdx.x * kTrsScan + e * kWG + threadIdx.x;
        if (i < n) h += trs_head(lower, i, rp, col, dpos);
    }
    h = wave_sum(h);
    if (threadIdx.x % kWave == 0) part[threadIdx.x / kWave] = h;
    __syncthreads();
    if (threadIdx.x == 0) sums[blockIdx.x] = part[0] + part[1] + part[2] + part[3];
}

// Inclusive sum over the workgroup's 256 threads.
__device__ __forceinline__ int trs_block_scan(int v, int *part) {
    const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const int u = __shfl_up(v, d, kWave);
        if (lane >= d) v += u;
    }
    __syncthreads();
    if (lane == kWave - 1) part[wid] = v;
    __syncthreads();
    for (int k = 0; k < wid; ++k) v += part[k];
    return v;
}

// Exclusive sums in place, a workgroup for each of two arrays; the total goes
// behind the last.
__global__ __launch_bounds__(kWG) void k_trs_scan(int n0, int *a0, int n1, int *a1) {
    __shared__ int part[kWG / kWave];
    __shared__ int carry;
    const int nb = blockIdx.y ? n1 : n0;
    int *sums = blockIdx.y ? a1 : a0;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int b0 = 0; b0 < nb; b0 += kWG) {
        const int b = b0 + threadIdx.x;
        const int v = b < nb ? sums[b] : 0;
        const int s = trs_block_scan(v, part) + carry;
        if (b < nb) sums[b] = s - v;
        __syncthreads();
        if (threadIdx.x == kWG - 1) carry = s;
        __syncthreads();
    }
    if (threadIdx.x == 0) sums[nb] = carry;
}

// Chain of every row and first row of every chain (cstart[nch] = n).  With one
// block of rows nothing is summed before: the total is found here.
__global__ __launch_bounds__(kWG) void k_trs_chains(int64_t n, const int *__restrict__ rp,
                                                    const int *__restrict__ col, const int *__restrict__ dpos,
                                                    TrsPair q, int nb) {
    __shared__ int part[kWG / kWave];
    __shared__ int carry;
    const bool lower = blockIdx.y == 0;
    int *sums = q.sums[blockIdx.y];
    int *rowchain = q.rowchain[blockIdx.y], *cstart = q.cstart[blockIdx.y];
    if (threadIdx.x == 0) carry = nb > 1 ? sums[blockIdx.x] : 0;
    __syncthreads();
    for (int e = 0; e < kTrsScan / kWG; ++e) {
        const int64_t i = (int64_t)blockIdx.x * kTrsScan + e * kWG + threadIdx.x;
        const int h = i < n ? (int)trs_head(lower, i, rp, col, dpos) : 0;
        const int s = trs_block_scan(h, part) + carry;
        if (i < n) {
            rowchain[i] = s - 1;
            if (h) cstart[s - 1] = (int)i;
        }
        __syncthreads();
        if (threadIdx.x == kWG - 1) carry = s;
        __syncthreads();
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (nb == 1) sums[1] = carry;
        cstart[sums[nb]] = (int)n;
    }
}

// Entries of row i's triangle besides the chain neighbour, in column order.
template <typename F>
__device__ __forceinline__ void trs_entries(bool lower, int i, const int *__restrict__ rp,
                                            const int *__restrict__ col, const int *__restrict__ dpos, F f) {
    const int q0 = lower ? rp[i] : dpos[i] + 1, q1 = lower ? dpos[i] : rp[i + 1];
    const int nb = lower ? i - 1 : i + 1;
    for (int q = q0; q < q1; ++q)
        if (col[q] != nb) f(q, col[q]);
}

__global__ __launch_bounds__(kWG) void k_trs_stats(int64_t n, const int *__restrict__ rp,
                                                   const int *__restrict__ col, const int *__restrict__ dpos,
                                                   TrsPair pr, int nb, TrsHead *h) {
    __shared__ int part[4][kWG / kWave];
    const bool lower = blockIdx.y == 0;
    const int *rowchain = pr.rowchain[blockIdx.y], *cstart = pr.cstart[blockIdx.y], *nchp = pr.sums[blockIdx.y] + nb;
    TrsInfo *f = h->f + blockIdx.y;
    int v[4] = {0, -INT_MAX, 0, 0};  // widest, -closest, farthest, longest
    // Columns are checked before they index anything: only validated matrices
    // are known to be canonical.
    int faults = 0;
    const int64_t nch = *nchp;
    for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < n; i += (int64_t)gridDim.x * kWG) {
        int a = 0, last = lower ? -1 : (int)i;
        const int me = rowchain[i];
        const int q0 = lower ? rp[i] : dpos[i] + 1, q1 = lower ? dpos[i] : rp[i + 1];
        for (int q = q0; q < q1; ++q) {
            const int c = col[q];
            if (c < 0 || c >= n) {
                faults |= kTrsOutside;
                continue;
            }
            if (c <= last || (lower && c >= (int)i)) faults |= kTrsUnsorted;
            last = c;
            if (c == (lower ? (int)i - 1 : (int)i + 1)) continue;  // the chain neighbour
            ++a;
            const int o = abs(me - rowchain[c]);
            if (o > 1) {
                v[1] = -o > v[1] ? -o : v[1];
                v[2] = o > v[2] ? o : v[2];
            }
        }
        v[0] = a > v[0] ? a : v[0];
        if (i < nch) {
            const int len = cstart[i + 1] - cstart[i];
            v[3] = len > v[3] ? len : v[3];
        }
    }
    // one atomic per workgroup and value: one per wave took 286 us on a 101^3 grid
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int m = wave_max(v[j]);
        if (threadIdx.x % kWave == 0) part[j][threadIdx.x / kWave] = m;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        const int *q = part[threadIdx.x];
        const int m = max(max(q[0], q[1]), max(q[2], q[3]));
        if (threadIdx.x == 0) atomicMax(&f->w, m);
        else if (threadIdx.x == 1) atomicMin(&f->lo, -m);
        else if (threadIdx.x == 2) atomicMax(&f->hi, m);
        else atomicMax(&f->longest, m);
    }
    if (faults) atomicOr(&f->faults, faults);
    if (blockIdx.x == 0 && threadIdx.x == 0) f->nch = (int)nch;
}

// f->bad = 1 when an operand's tile is not at or before its row's tile in
// both tile coordinates: then a row's operands always come from tiles with
// earlier tickets, in ascending order for L and descending for U.
__global__ void k_trs_order(int64_t n, const int *__restrict__ rp, const int *__restrict__ col,
                            const int *__restrict__ dpos, TrsPair q, TrsHead *h) {
    const bool lower = blockIdx.y == 0;
    const int *rowchain = q.rowchain[blockIdx.y];
    TrsInfo *f = h->f + blockIdx.y;
    const TrsPlan p = trs_plan(n, *f);
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n || !p.ok || p.W == 0) return;
    auto tj = [&](int t) { return (t % p.W + (int64_t)p.skew * (t / p.W)) / kTrsTJ; };
    auto tk = [&](int t) { return (t / p.W) / p.TK; };
    const int me = rowchain[i];
    bool wrong = false;
    trs_entries(lower, (int)i, rp, col, dpos, [&](int, int c) {
        const int ot = rowchain[c];
        const int first = lower ? ot : me, then = lower ? me : ot;
        wrong = wrong || tj(first) > tj(then) || tk(first) > tk(then);
    });
    if (__any(wrong) && threadIdx.x % kWave == 0) atomicOr(&f->bad, 1);
}

// The packing of a triangle: its plan, the temporaries (rowchain, first, cgroup)
// and the solve's arrays.
struct TrsPacked {
    TrsPlan p;
    int nch, w, cap;
    const int *rowchain, *first;  // first: the chains' first rows
    int *cgroup, *cstart, *gptr, *glist, *cbase, *code;
    double *val, *prev, *diag;
};

__global__ void k_trs_sizes(TrsPacked lo, TrsPacked up) {
    const TrsPacked &T = blockIdx.y ? up : lo;
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= T.p.groups) return;
    int c = 0;
    trs_group(T.p, T.nch, g, [&](int) { ++c; });
    T.gptr[g] = c;
}

// Each group's chains, their places (one after the other) and their group.  SUM:
// one wave holds all groups and sums their sizes itself.
template <bool SUM>
__global__ __launch_bounds__(kWave) void k_trs_lists(TrsPacked lo, TrsPacked up) {
    const TrsPacked &T = blockIdx.y ? up : lo;
    const int g = blockIdx.x * kWave + threadIdx.x;
    int q = 0;
    if (SUM) {
        int c = 0;
        if (g < T.p.groups) trs_group(T.p, T.nch, g, [&](int) { ++c; });
        int end = c;
        for (int d = 1; d < kWave; d <<= 1) {
            const int u = __shfl_up(end, d, kWave);
            if (g >= d) end += u;
        }
        q = end - c;
        if (g < T.p.groups) {
            T.gptr[g] = q;
            if (g == T.p.groups - 1) T.gptr[g + 1] = end;
        }
    }
    if (g >= T.p.groups) return;
    if (!SUM) q = T.gptr[g];
    int64_t rows = 0;
    trs_group(T.p, T.nch, g, [&](int t) {
        T.glist[q++] = t;
        T.cbase[t] = (int)(rows < INT_MAX ? rows : INT_MAX);
        T.cgroup[t] = g;
        rows += T.first[t + 1] - T.first[t];
    });
}

__global__ void k_trs_encode(int64_t n, int64_t n_pad, const int *__restrict__ rp, const int *__restrict__ col,
                             const int *__restrict__ dpos, const double *__restrict__ lu, TrsPacked lo, TrsPacked up,
                             unsigned *tickets) {
    const bool lower = blockIdx.y == 0;
    const TrsPacked &T = lower ? lo : up;
    const int *__restrict__ rowchain = T.rowchain, *__restrict__ cstart = T.first, *__restrict__ cgroup = T.cgroup,
                            *__restrict__ cbase = T.cbase;
    int *__restrict__ code = T.code;
    double *__restrict__ val = T.val;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (lower && i < 3) tickets[i] = 0;
    if (i <= T.nch) T.cstart[i] = cstart[i];
    if (i >= n) return;
    const int g = cgroup[rowchain[i]], w = T.w, cap = T.cap;
    int a = 0;
    trs_entries(lower, (int)i, rp, col, dpos, [&](int q, int c) {
        const int t = rowchain[c];
        int e = c;
        if (cgroup[t] == g) {
            const int64_t pl = (int64_t)cbase[t] + (lower ? c - cstart[t] : cstart[t + 1] - 1 - c);
            if (pl < cap) e = (int)((unsigned)pl | 0x80000000u);
        }
        code[(int64_t)a * n_pad + i] = e;
        val[(int64_t)a * n_pad + i] = lu[q];
        ++a;
    });
    for (; a < w; ++a) {
        code[(int64_t)a * n_pad + i] = kTrsPad;
        val[(int64_t)a * n_pad + i] = 0.0;
    }
    const int nbq = lower ? dpos[i] - 1 : dpos[i] + 1;
    const bool has = lower ? nbq >= rp[i] && col[nbq] == (int)i - 1 : nbq < rp[i + 1] && col[nbq] == (int)i + 1;
    T.prev[i] = has ? lu[nbq] : 0.0;
    if (!lower) T.diag[i] = lu[dpos[i]];
}

namespace {

unsigned trs_grid(int64_t n, int per) { return (unsigned)((n + per - 1) / per > 0 ? (n + per - 1) / per : 1); }

#define TRS_TRY(expr, what)                                                                                    \
    do {                                                                                                       \
        const hipError_t e_ = (expr);                                                                          \
        if (e_ != hipSuccess) return set_error(MXL_ERR_DEVICE, std::string(what ": ") + hipGetErrorString(e_)); \
    } while (0)

template <int NE, int RD>
hipError_t trs_allow_lds() {
    const int v = (int)kTrsLdsMax;
    hipError_t e = hipFuncSetAttribute((const void *)k_trs_chain<true, NE, kTrsLoaders, RD>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, v);
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void *)k_trs_chain<false, NE, kTrsLoaders, RD>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, v);
    return e;
}

TrsView trs_view(const IluImpl &P, const TrsSide &T, bool lower) {
    TrsView M;
    M.n_pad = P.n_pad;
    M.code = (const int *)T.code->p;
    M.val = (const double *)T.val->p;
    M.prev = (const double *)T.prev->p;
    M.diag = lower ? nullptr : (const double *)P.udiag->p;
    M.w = T.w;
    M.cstart = (const int *)T.cstart->p;
    M.cbase = (const int *)T.cbase->p;
    M.glist = (const int *)T.glist->p;
    M.gptr = (const int *)T.gptr->p;
    M.groups = T.groups;
    M.C = T.C;
    M.cap = T.cap;
    M.fail = lower ? 2 : 1;
    M.passes = P.wait_passes;
    return M;
}

template <bool LOWER, int NE, int RD>
void trs_launch(const TrsView &M, const double *b, double *x, double *znext, double alpha, double beta, double *out,
                unsigned *ticket, hipStream_t s) {
    hipLaunchKernelGGL((k_trs_chain<LOWER, NE, kTrsLoaders, RD>), dim3(M.groups), dim3(kTrsLanes + kTrsLoaders),
                       (trs_lds_bytes<LOWER, NE, kTrsLoaders, RD>(M.cap)), s, M, b, x, znext, alpha, beta, out, ticket);
}

}  // namespace

namespace {
struct TrsBoth {
    TrsInfo f[2];
    TrsPlan p[2];
};
}  // namespace

size_t chain_head_bytes() { return sizeof(TrsHead); }

hipError_t chain_head_init(const BufPtr &head, int *&bad, int *&widths, hipStream_t s) {
    auto *h = (TrsHead *)head->p;
    bad = &h->bad;
    widths = h->widths;
    hipLaunchKernelGGL(k_ilu_begin, dim3(1), dim3(64), 0, s, h);
    return hipGetLastError();
}

void chain_plan_want(ChainPlan &C, int64_t n, Arena &tmp) {
    for (int k = 0; k < 2; ++k) {
        tmp.want(C.sums[k], ((size_t)trs_grid(n, kTrsScan) + 1) * 4);
        tmp.want(C.rowchain[k], (size_t)n * 4);
        tmp.want(C.cstart[k], (size_t)(n + 1) * 4);
        tmp.want(C.cgroup[k], (size_t)n * 4);
    }
}

// The device passes of the plan.  Rows without a diagonal (the caller's to
// report) are read in bounds.
hipError_t chain_gather(const IluImpl &P, const ChainPlan &C, const BufPtr &head) {
    const MatrixImpl &A = *P.A;
    const int64_t n = A.nrows;
    hipStream_t s = A.ctx->stream;
    const int *rp = (const int *)A.row_ptr->p, *col = (const int *)A.col->p, *dpos = (const int *)P.dpos->p;
    const int nb = (int)trs_grid(n, kTrsScan);
    TrsPair q;
    for (int k = 0; k < 2; ++k) {
        q.sums[k] = (int *)C.sums[k]->p;
        q.rowchain[k] = (int *)C.rowchain[k]->p;
        q.cstart[k] = (int *)C.cstart[k]->p;
    }
    auto *h = (TrsHead *)head->p;
    if (nb > 1) {
        hipLaunchKernelGGL(k_trs_count, dim3(nb, 2), dim3(kWG), 0, s, n, rp, col, dpos, q);
        hipLaunchKernelGGL(k_trs_scan, dim3(1, 2), dim3(kWG), 0, s, nb, q.sums[0], nb, q.sums[1]);
    }
    hipLaunchKernelGGL(k_trs_chains, dim3(nb, 2), dim3(kWG), 0, s, n, rp, col, dpos, q, nb);
    hipLaunchKernelGGL(k_trs_stats, dim3(std::min(trs_grid(n, kWG), 1024u), 2), dim3(kWG), 0, s, n, rp, col, dpos, q, nb,
                       h);
    hipLaunchKernelGGL(k_trs_order, dim3(trs_grid(n, 256), 2), dim3(256), 0, s, n, rp, col, dpos, q, h);
    return hipGetLastError();
}

// Reads the head: bad and, where a plan was gathered (ok), whether the chains suit.
mxl_status chain_read(const IluImpl &P, ChainPlan &C, const BufPtr &head, int &bad, bool &ok) {
    const int64_t n = P.A->nrows;
    hipStream_t s = P.A->ctx->stream;
    TrsHead hh;
    TRS_TRY(hipMemcpyAsync(&hh, head->p, sizeof hh, hipMemcpyDeviceToHost, s), "ILU set-up");
    TRS_TRY(hipStreamSynchronize(s), "ILU set-up");
    bad = hh.bad;
    const bool gathered = ok;
    ok = false;
    if (!gathered || bad != INT_MAX) return MXL_OK;
    auto both = std::make_shared<TrsBoth>();
    TrsInfo *f = both->f;
    TrsPlan *p = both->p;
    f[0] = hh.f[0];
    f[1] = hh.f[1];
    if ((f[0].faults | f[1].faults) & kTrsOutside)
        return set_error(MXL_ERR_INVALID_MATRIX, "a column index lies outside the matrix");
    for (int k = 0; k < 2; ++k) {
        p[k] = trs_plan(n, f[k]);
        if (!p[k].ok) return MXL_OK;
        if (f[k].bad) {
            p[k].W = 0;
            trs_count_groups(p[k], f[k].nch);
        }
    }
    // Every row is padded to the widest one.  The line is the level layout's, which
    // counts the neighbour among a row's entries: above it one wide row among short ones
    // would multiply the factors' memory (a row of 12 entries on either side in a
    // tridiagonal matrix: 288 bytes a row beside 36) and every application's reads.
    const int64_t n_pad = (n + 63) / 64 * 64;
    if ((int64_t)(f[0].w + f[1].w + 2) * n_pad > 4 * P.A->nnz + 2 * n) return MXL_OK;
    C.both = both;
    ok = true;
    return MXL_OK;
}

size_t chain_want(IluImpl &P, const ChainPlan &C, Arena &keep) {
    const int64_t n = P.A->nrows;
    const TrsBoth &B = *(const TrsBoth *)C.both.get();
    P.n_pad = (n + 63) / 64 * 64;
    size_t bytes = 0;
    auto want = [&](BufPtr &b, size_t sz) {
        keep.want(b, sz);
        bytes += sz;
    };
    for (int k = 0; k < 2; ++k) {
        TrsSide &T = k == 0 ? P.lo : P.up;
        T.groups = B.p[k].groups;
        T.C = B.p[k].C;
        T.w = B.f[k].w;
        T.cap = (int)std::min<int64_t>((int64_t)B.p[k].C * B.f[k].longest, B.p[k].places);
        want(T.code, (size_t)T.w * P.n_pad * 4);
        want(T.cstart, (size_t)(B.f[k].nch + 1) * 4);
        want(T.cbase, (size_t)B.f[k].nch * 4);
        want(T.glist, (size_t)B.f[k].nch * 4);
        want(T.gptr, (size_t)(B.p[k].groups + 1) * 4);
        want(T.val, (size_t)T.w * P.n_pad * 8);
        want(T.prev, (size_t)n * 8);
    }
    want(P.udiag, (size_t)n * 8);
    return bytes;
}

mxl_status chain_pack(IluImpl &P, const ChainPlan &C) {
    const MatrixImpl &A = *P.A;
    const int64_t n = A.nrows;
    hipStream_t s = A.ctx->stream;
    const TrsBoth &B = *(const TrsBoth *)C.both.get();
    TrsPacked t[2];
    for (int k = 0; k < 2; ++k) {
        const TrsSide &T = k == 0 ? P.lo : P.up;
        t[k] = {B.p[k], B.f[k].nch, T.w, T.cap, (const int *)C.rowchain[k]->p, (const int *)C.cstart[k]->p,
                (int *)C.cgroup[k]->p, (int *)T.cstart->p, (int *)T.gptr->p, (int *)T.glist->p, (int *)T.cbase->p,
                (int *)T.code->p, (double *)T.val->p, (double *)T.prev->p, (double *)P.udiag->p};
    }
    const dim3 g(trs_grid(std::max(t[0].p.groups, t[1].p.groups), kWave), 2);
    if (g.x == 1) {
        hipLaunchKernelGGL(k_trs_lists<true>, g, dim3(kWave), 0, s, t[0], t[1]);
    } else {
        hipLaunchKernelGGL(k_trs_sizes, g, dim3(kWave), 0, s, t[0], t[1]);
        hipLaunchKernelGGL(k_trs_scan, dim3(1, 2), dim3(kWG), 0, s, t[0].p.groups, t[0].gptr, t[1].p.groups, t[1].gptr);
        hipLaunchKernelGGL(k_trs_lists<false>, g, dim3(kWave), 0, s, t[0], t[1]);
    }
    hipLaunchKernelGGL(k_trs_encode, dim3(trs_grid(n + 1, 256), 2), dim3(256), 0, s, n, P.n_pad,
                       (const int *)A.row_ptr->p, (const int *)A.col->p, (const int *)P.dpos->p,
                       (const double *)P.lu->p, t[0], t[1], (unsigned *)P.tickets->p);
    TRS_TRY(hipGetLastError(), "triangular solve factors");
    TRS_TRY((trs_allow_lds<kTrsNarrow, 2>()), "LDS attribute");
    TRS_TRY((trs_allow_lds<kTrsWide, 1>()), "LDS attribute");
    P.wait_passes = trs_wait_passes(n);
    TRS_TRY(hipStreamSynchronize(s), "triangular solve factors");  // the plan's temporaries end here
    P.chain = true;
    return MXL_OK;
}

mxl_status ilu_chain_check(const IluImpl &P) {
    hipStream_t s = P.A->ctx->stream;
    unsigned gave_up = 0;
    TRS_TRY(hipMemcpyAsync(&gave_up, (unsigned *)P.tickets->p + 2, 4, hipMemcpyDeviceToHost, s), "triangular solve");
    TRS_TRY(hipStreamSynchronize(s), "triangular solve");
    if (!gave_up) return MXL_OK;
    hipLaunchKernelGGL(k_trs_clear, dim3(1), dim3(64), 0, s, (unsigned *)P.tickets->p);  // reported once
    return set_error(MXL_ERR_INTERNAL, "a triangular solve gave up waiting for its operands; its result holds NaN");
}

hipError_t ilu_chain_apply(const IluImpl &P, double alpha, const double *r, double beta, double *out, hipStream_t s) {
    const int64_t n = P.A->nrows;
    double *y = (double *)P.y->p, *z = (double *)P.z->p;
    unsigned *tk = (unsigned *)P.tickets->p;
    const TrsView L = trs_view(P, P.lo, true), U = trs_view(P, P.up, false);
    hipLaunchKernelGGL(k_trs_begin, dim3(trs_grid(n, 256)), dim3(256), 0, s, n, y, tk);
    if (L.w > kTrsNarrow) trs_launch<true, kTrsWide, 1>(L, r, y, z, 1.0, 0.0, nullptr, tk, s);
    else trs_launch<true, kTrsNarrow, 2>(L, r, y, z, 1.0, 0.0, nullptr, tk, s);
    if (U.w > kTrsNarrow) trs_launch<false, kTrsWide, 1>(U, y, z, nullptr, alpha, beta, out, tk + 1, s);
    else trs_launch<false, kTrsNarrow, 2>(U, y, z, nullptr, alpha, beta, out, tk + 1, s);
    return hipGetLastError();
}

// Not an entry point: lets a test make the solves of P give up after `passes`
// passes without progress.
int ilu_chain_set_wait_passes(mxl_op *P, int64_t passes) {
    if (!P || P->kind != MXL_OP_ILU || !P->ilu->chain || passes < 0) return 1;
    P->ilu->wait_passes = passes;
    return 0;
}

}  // namespace mxl
