// batched.hip -- thousands of independent small Jacobi-PCG solves in one call
// (per-system stopping status: the per-right-hand-side stopping status of the
// criteria in Sec. 2.5 of the paper, applied to independent systems), and the
// one-workgroup solves of a single small system.
//
// Design (gfx950), two ways.  By size classes, the way of a call without a
// schedule: systems of at most 1,024 rows and kClsW entries a row are sorted
// by size, and a workgroup a system holds matrix and vectors in registers
// (k_batch_pcg_cls); the others run beside the classes by the second way.
// Persistent kernels, the way of a chosen schedule, of a batch that has no ELL
// copy and of those other systems: a grid of wgs_per_cu x num_CU workgroups
// stays resident;
// each workgroup pulls a system id from an atomic queue, runs the whole CG
// for that system with its vectors r, p, q, x in LDS (or in a per-workgroup
// global scratch slice when the system is too large for LDS), reduces dot
// products inside the workgroup (fixed tree: deterministic), writes x, the
// iteration count, the recurrence residual and the stop reason, and pulls
// the next id.  Every workgroup exits when the queue is drained.  The
// schedule (workgroup size, residency, order) can be chosen by an autotuner
// that times the candidates, and the size classes, on the actual batch.
#include <algorithm>
#include <chrono>
#include <climits>
#include <cmath>
#include <cstring>
#include <map>
#include <mutex>
#include <numeric>
#include <string>
#include <vector>

#include "device_common.hpp"
#include "internal.hpp"

namespace mxl {

struct BatchImpl {
    CtxRef ctx;
    int64_t nsys = 0, rows = 0, nnz = 0;
    std::vector<int32_t> sys_ptr_h;
    int max_n = 0;
    BufPtr sys_ptr, row_ptr, col, val;
    BufPtr dinv;             // FP64 1/a_ii of every row
    BufPtr order_input, order_big;  // processing orders
    BufPtr queue;            // uint32 work counter
    BufPtr scratch;          // per-workgroup vectors for systems larger than LDS
    int64_t scratch_elems = 0;
    bool tuned = false;
    mxl_tuning best{};
    int small_shape = -1;    // single-system register-cached shape (-1: not chosen)
    int small_bi_shape = -1; // the same for the one-workgroup BiCGSTAB
    // Per-system slot-major ELL copy (built when it is compact): system s has
    // w_s = its longest row; slot e of local row i is at off_s + e*n_s + i,
    // columns as int16 local indices, -1 for padding.
    bool ell = false;
    int w_max = 0;
    int64_t ell_slots = 0;
    BufPtr ell_val, ell_col, ell_off, ell_w;
    // The size-class schedule (with the ELL copy): systems a workgroup can
    // hold in registers, by class and largest first, and the others.
    BufPtr desc, order_rest;     // order_rest: the others in input order, then largest first
    int64_t cls_begin[6] = {0};  // class k: desc[cls_begin[k]] .. desc[cls_begin[k + 1] - 1]
    int64_t nrest = 0;
    bool cls_best = true;        // the schedule of calls without one (autotuning may find another faster)
    // the others run beside the classes (batches with both)
    hipStream_t side = nullptr;
    hipEvent_t fork = nullptr, join = nullptr;
    BatchImpl() = default;
    BatchImpl(const BatchImpl &) = delete;
    BatchImpl &operator=(const BatchImpl &) = delete;
    ~BatchImpl() {
        if (fork) (void)hipEventDestroy(fork);
        if (join) (void)hipEventDestroy(join);
        if (side) (void)hipStreamDestroy(side);
    }
};

// One system of the size-class schedule.
struct BatchDesc {
    int32_t sys, r0, n, w;
    int64_t off;
    int64_t pad;
};
constexpr int kClsN[5] = {64, 128, 256, 512, 1024};  // rows of the classes
constexpr int kClsR[5] = {1, 2, 2, 2, 2};            // rows per thread
constexpr int kClsW = 28;                            // entries per row held in registers

template <int B>
__device__ __forceinline__ double wg_sum(double v, double *red) {
    constexpr int NW = B / kWave;
    v = wave_sum(v);
    if (NW == 1) return v;
    const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
    __syncthreads();
    if (lane == 0) red[wid] = v;
    __syncthreads();
    double a = red[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) a += red[w];
    return a;
}

template <int B>
__device__ __forceinline__ void wg_sum2(double &u, double &v, double *red) {
    constexpr int NW = B / kWave;
    u = wave_sum(u);
    v = wave_sum(v);
    if (NW == 1) return;
    const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
    __syncthreads();
    if (lane == 0) {
        red[wid] = u;
        red[NW + wid] = v;
    }
    __syncthreads();
    double a = red[0], c = red[NW];
#pragma unroll
    for (int w = 1; w < NW; ++w) {
        a += red[w];
        c += red[NW + w];
    }
    u = a;
    v = c;
}

template <int B>
__global__ __launch_bounds__(B) void k_batch_pcg(
    int64_t nsys, const int *__restrict__ sys_ptr, const int *__restrict__ rp,
    const int *__restrict__ col, const double *__restrict__ val, const double *__restrict__ dinv,
    const double *__restrict__ bvec, double *__restrict__ xout, int *__restrict__ iters_out,
    double *__restrict__ rel_out, uint8_t *__restrict__ status_out, const int *__restrict__ order,
    unsigned *__restrict__ queue, double red_factor, int64_t max_iters_fixed, int iter_factor,
    int chk, int lds_cap, double *__restrict__ scratch, int64_t scratch_stride, int use_x0) {
    extern __shared__ double smem[];
    __shared__ double red[2 * (B / kWave)];
    __shared__ int s_q;
    const int tid = threadIdx.x;
    for (;;) {
        if (tid == 0) s_q = (int)atomicAdd(queue, 1u);
        __syncthreads();
        const int qi = s_q;
        __syncthreads();
        if ((int64_t)qi >= nsys) break;
        const int s = order[qi];
        const int r0 = sys_ptr[s];
        const int n = sys_ptr[s + 1] - r0;
        const bool in_lds = n <= lds_cap;
        double *base = in_lds ? smem : scratch + (int64_t)blockIdx.x * scratch_stride;
        double *x = base, *r = base + n, *p = base + 2 * n, *q = base + 3 * n;
        const double *b = bvec + r0;
        const double *di = dinv + r0;
        const int *rps = rp + r0;
        // x = x0 (or 0), r = b - A x, p = z = D^{-1} r
        for (int i = tid; i < n; i += B) x[i] = use_x0 ? xout[r0 + i] : 0.0;
        if (use_x0) __syncthreads();
        double rz = 0.0, rr0 = 0.0, bb = 0.0;
        for (int i = tid; i < n; i += B) {
            const double bi = b[i];
            double ax = 0.0;
            if (use_x0)
                for (int e = rps[i]; e < rps[i + 1]; ++e) ax += val[e] * x[col[e]];
            const double ri = bi - ax;
            const double zi = di[i] * ri;
            r[i] = ri;
            p[i] = zi;
            rz += ri * zi;
            rr0 += ri * ri;
            bb += bi * bi;
        }
        wg_sum2<B>(rz, bb, red);
        rr0 = wg_sum<B>(rr0, red);
        const double nb = sqrt(bb);
        const int64_t maxit = max_iters_fixed > 0 ? max_iters_fixed : (int64_t)iter_factor * n;
        int stop = ST_RUN;
        int64_t k = 0;
        double rr = rr0;
        if (bb == 0.0) {  // zero right-hand side: x = 0
            for (int i = tid; i < n; i += B) x[i] = 0.0;
            stop = ST_CONVERGED;
        } else if (sqrt(rr) <= red_factor * nb) {
            stop = ST_CONVERGED;
        }
        double rho = rz;
        while (stop == ST_RUN && k < maxit) {
            __syncthreads();  // p complete
            double pq = 0.0;
            for (int i = tid; i < n; i += B) {
                const int e0 = rps[i], e1 = rps[i + 1];
                double acc = 0.0;
                for (int e = e0; e < e1; ++e) acc += val[e] * p[col[e]];
                q[i] = acc;
                pq += p[i] * acc;
            }
            const double eta = wg_sum<B>(pq, red);
            if (chk && !finite_d(eta)) { stop = ST_NONFINITE; break; }
            if (eta <= 0.0) { stop = ST_BREAKDOWN; break; }
            const double alpha = rho / eta;
            double rzn = 0.0, rrn = 0.0;
            for (int i = tid; i < n; i += B) {
                x[i] += alpha * p[i];
                const double ri = r[i] - alpha * q[i];
                r[i] = ri;
                rzn += ri * (di[i] * ri);
                rrn += ri * ri;
            }
            wg_sum2<B>(rzn, rrn, red);
            ++k;
            rr = rrn;
            if (chk && !finite_d(rr)) { stop = ST_NONFINITE; break; }
            if (sqrt(rr) <= red_factor * nb) { stop = ST_CONVERGED; break; }
            if (chk && !finite_d(rzn)) { stop = ST_NONFINITE; break; }
            if (rzn == 0.0) { stop = ST_BREAKDOWN; break; }
            const double beta = rzn / rho;
            rho = rzn;
            for (int i = tid; i < n; i += B) p[i] = di[i] * r[i] + beta * p[i];
        }
        if (stop == ST_RUN) stop = ST_MAX_ITERS;
        __syncthreads();
        for (int i = tid; i < n; i += B) xout[r0 + i] = x[i];
        if (tid == 0) {
            iters_out[s] = (int)k;
            rel_out[s] = nb > 0.0 ? sqrt(rr) / nb : 0.0;
            status_out[s] = (uint8_t)stop;
        }
        __syncthreads();
    }
}

// The same persistent Jacobi-PCG on the per-system ELL copy.  A system
// whose five vectors (x, r, p, q, dinv) fit the workgroup's LDS budget keeps
// them there, and its matrix too when that also fits, so every iteration
// after the first reads only LDS; the product walks slot-major entries
// (consecutive rows at consecutive addresses) in each row's stored order,
// so q and every scalar equal k_batch_pcg's at the same workgroup size.
// Larger systems keep their vectors in a global scratch slice and read the
// matrix from the global ELL copy.
template <int B>
__global__ __launch_bounds__(B) void k_batch_pcg_ell(
    int64_t nsys, const int *__restrict__ sys_ptr, const int64_t *__restrict__ ell_off,
    const int *__restrict__ ell_w, const double *__restrict__ ell_val, const short *__restrict__ ell_col,
    const double *__restrict__ dinv, const double *__restrict__ bvec, double *__restrict__ xout,
    int *__restrict__ iters_out, double *__restrict__ rel_out, uint8_t *__restrict__ status_out,
    const int *__restrict__ order, unsigned *__restrict__ queue, double red_factor, int64_t max_iters_fixed,
    int iter_factor, int chk, int64_t lds_budget, double *__restrict__ scratch, int64_t scratch_stride,
    int use_x0) {
    extern __shared__ double smem[];
    __shared__ double red[2 * (B / kWave)];
    __shared__ int s_q;
    const int tid = threadIdx.x;
    for (;;) {
        if (tid == 0) s_q = (int)atomicAdd(queue, 1u);
        __syncthreads();
        const int qi = s_q;
        __syncthreads();
        if ((int64_t)qi >= nsys) break;
        const int s = order[qi];
        const int r0 = sys_ptr[s];
        const int n = sys_ptr[s + 1] - r0;
        const int w = ell_w[s];
        const int64_t off = ell_off[s];
        const int64_t vec_bytes = (int64_t)40 * n, mat_bytes = (int64_t)10 * w * n;
        const bool in_lds = vec_bytes <= lds_budget;
        const bool mat_lds = in_lds && vec_bytes + mat_bytes <= lds_budget;
        double *base = in_lds ? smem : scratch + (int64_t)blockIdx.x * scratch_stride;
        double *x = base, *r = base + n, *p = base + 2 * n, *q = base + 3 * n, *di = base + 4 * n;
        const double *Vm = mat_lds ? base + 5 * n : ell_val + off;
        const short *Cm = mat_lds ? (const short *)(base + 5 * n + (int64_t)w * n) : ell_col + off;
        if (mat_lds) {
            double *vl = base + 5 * n;
            short *cl = (short *)(base + 5 * n + (int64_t)w * n);
            for (int64_t j = tid; j < (int64_t)w * n; j += B) {
                vl[j] = ell_val[off + j];
                cl[j] = ell_col[off + j];
            }
        }
        const double *b = bvec + r0;
        for (int i = tid; i < n; i += B) {
            x[i] = use_x0 ? xout[r0 + i] : 0.0;
            di[i] = dinv[r0 + i];
        }
        __syncthreads();
        // r = b - A x, p = z = D^{-1} r
        double rz = 0.0, rr0 = 0.0, bb = 0.0;
        for (int i = tid; i < n; i += B) {
            const double bi = b[i];
            double ax = 0.0;
            if (use_x0)
                for (int e = 0; e < w; ++e) {
                    const int c = Cm[(int64_t)e * n + i];
                    if (c >= 0) ax += Vm[(int64_t)e * n + i] * x[c];
                }
            const double ri = bi - ax;
            const double zi = di[i] * ri;
            r[i] = ri;
            p[i] = zi;
            rz += ri * zi;
            rr0 += ri * ri;
            bb += bi * bi;
        }
        wg_sum2<B>(rz, bb, red);
        rr0 = wg_sum<B>(rr0, red);
        const double nb = sqrt(bb);
        const int64_t maxit = max_iters_fixed > 0 ? max_iters_fixed : (int64_t)iter_factor * n;
        int stop = ST_RUN;
        int64_t k = 0;
        double rr = rr0;
        if (bb == 0.0) {  // zero right-hand side: x = 0
            for (int i = tid; i < n; i += B) x[i] = 0.0;
            stop = ST_CONVERGED;
        } else if (sqrt(rr) <= red_factor * nb) {
            stop = ST_CONVERGED;
        }
        double rho = rz;
        while (stop == ST_RUN && k < maxit) {
            __syncthreads();  // p complete
            double pq = 0.0;
            for (int i = tid; i < n; i += B) {
                double acc = 0.0;
#pragma unroll 4
                for (int e = 0; e < w; ++e) {
                    const int c = Cm[(int64_t)e * n + i];
                    if (c >= 0) acc += Vm[(int64_t)e * n + i] * p[c];
                }
                q[i] = acc;
                pq += p[i] * acc;
            }
            const double eta = wg_sum<B>(pq, red);
            if (chk && !finite_d(eta)) { stop = ST_NONFINITE; break; }
            if (eta <= 0.0) { stop = ST_BREAKDOWN; break; }
            const double alpha = rho / eta;
            double rzn = 0.0, rrn = 0.0;
            for (int i = tid; i < n; i += B) {
                x[i] += alpha * p[i];
                const double ri = r[i] - alpha * q[i];
                r[i] = ri;
                rzn += ri * (di[i] * ri);
                rrn += ri * ri;
            }
            wg_sum2<B>(rzn, rrn, red);
            ++k;
            rr = rrn;
            if (chk && !finite_d(rr)) { stop = ST_NONFINITE; break; }
            if (sqrt(rr) <= red_factor * nb) { stop = ST_CONVERGED; break; }
            if (chk && !finite_d(rzn)) { stop = ST_NONFINITE; break; }
            if (rzn == 0.0) { stop = ST_BREAKDOWN; break; }
            const double beta = rzn / rho;
            rho = rzn;
            for (int i = tid; i < n; i += B) p[i] = di[i] * r[i] + beta * p[i];
        }
        if (stop == ST_RUN) stop = ST_MAX_ITERS;
        __syncthreads();
        for (int i = tid; i < n; i += B) xout[r0 + i] = x[i];
        if (tid == 0) {
            iters_out[s] = (int)k;
            rel_out[s] = nb > 0.0 ? sqrt(rr) / nb : 0.0;
            status_out[s] = (uint8_t)stop;
        }
        __syncthreads();
    }
}

// Sums over lanes by moves inside the vector unit (a shuffle through LDS
// costs about 100 cycles a step): lanes of a 16-lane row are rotated, rows
// and halves of the wave exchanged.  Every step adds the same two values in
// both partners, so all lanes end with the same bits.
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
constexpr int kDppXor1 = 0xB1, kDppRor1 = 0x121, kDppRor2 = 0x122, kDppRor4 = 0x124, kDppRor8 = 0x128;
// v plus its value 16 (HALF: 32) lanes away
template <bool HALF>
__device__ __forceinline__ double swap_add(double v) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned l = (unsigned)b, h = (unsigned)(b >> 32);
    unsigned l0, l1, h0, h1;
    if constexpr (HALF) {
        const auto x = __builtin_amdgcn_permlane32_swap(l, l, false, false);
        const auto y = __builtin_amdgcn_permlane32_swap(h, h, false, false);
        l0 = x[0]; l1 = x[1]; h0 = y[0]; h1 = y[1];
    } else {
        const auto x = __builtin_amdgcn_permlane16_swap(l, l, false, false);
        const auto y = __builtin_amdgcn_permlane16_swap(h, h, false, false);
        l0 = x[0]; l1 = x[1]; h0 = y[0]; h1 = y[1];
    }
    return __longlong_as_double((long long)((unsigned long long)h0 << 32 | l0)) +
           __longlong_as_double((long long)((unsigned long long)h1 << 32 | l1));
}

// Sum over the B-thread workgroup (at most 16 waves), in every thread; red:
// B / 64 doubles not in use by another sum since the barrier before the last one.
template <int B>
__device__ __forceinline__ double cls_sum(double v, double *red) {
    constexpr int NW = B / kWave;
    v += dpp_move<kDppRor8>(v);
    v += dpp_move<kDppRor4>(v);
    v += dpp_move<kDppRor2>(v);
    v += dpp_move<kDppXor1>(v);
    v = swap_add<true>(swap_add<false>(v));
    if constexpr (NW > 1) {
        const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
        if (lane == 0) red[wid] = v;
        __syncthreads();
        v = red[lane % NW];
        if constexpr (NW > 8) v += dpp_move<kDppRor8>(v);
        if constexpr (NW > 4) v += dpp_move<kDppRor4>(v);
        if constexpr (NW > 2) v += dpp_move<kDppRor2>(v);
        v += dpp_move<kDppRor1>(v);
    }
    return v;
}

// Two sums at once: after one exchange even lanes carry u and odd lanes v, so
// the two cost little more than one.  red: B / 32 doubles.
template <int B>
__device__ __forceinline__ void cls_sum2(double &u, double &v, double *red) {
    constexpr int NW = B / kWave;
    const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
    const bool odd = lane & 1;
    double t = odd ? v : u;
    t += dpp_move<kDppXor1>(odd ? u : v);
    t += dpp_move<kDppRor8>(t);
    t += dpp_move<kDppRor4>(t);
    t += dpp_move<kDppRor2>(t);
    t = swap_add<true>(swap_add<false>(t));
    if constexpr (NW > 1) {
        if (lane < 2) red[2 * wid + lane] = t;
        __syncthreads();
        t = red[lane % (2 * NW)];
        if constexpr (NW > 8) t = swap_add<false>(t);
        if constexpr (NW > 4) t += dpp_move<kDppRor8>(t);
        if constexpr (NW > 2) t += dpp_move<kDppRor4>(t);
        t += dpp_move<kDppRor2>(t);
    }
    const double o = dpp_move<kDppXor1>(t);
    u = odd ? o : t;
    v = odd ? t : o;
}

// The largest rr with sqrt(rr) <= tol, so that a criterion on the norm is one
// compare; ok = false where tol^2 leaves the normal range.
__device__ __forceinline__ double norm2_bound(double tol, bool &ok) {
    double top = tol * tol;
    ok = top > 1e-290 && top < 1e290;
    if (ok) {
        while (sqrt(top) > tol) top = __longlong_as_double(__double_as_longlong(top) - 1);
        for (double up = __longlong_as_double(__double_as_longlong(top) + 1); sqrt(up) <= tol;
             up = __longlong_as_double(__double_as_longlong(up) + 1))
            top = up;
    }
    return top;
}

// Jacobi-PCG of the systems of one size class, a workgroup each, with nothing
// but p outside the registers: a thread holds its one or two rows of the
// matrix (at most kClsW entries, two 16-bit LDS offsets to a register), of x,
// r, p and 1/a_ii, so an iteration reads p from LDS, reduces twice and touches
// no memory.  The matrices are read once.
//
// What bounds it: vector instructions (an FMA, an LDS address and a share of
// two reductions per entry) and the latency of an iteration's three barriers,
// with two waves per SIMD (28 entries of two rows take 244 registers).  Two
// rows per thread halve what every wave repeats (reductions, quotients):
// 730 -> 610 us for 10,000 banded systems of 32 to 1,024 rows, widths 5 to 27;
// reductions by lane moves instead of LDS shuffles and eight LDS reads under
// way: 610 -> 553 us (156 us of it is the one pass over the matrices, 20 us an
// iteration).  The persistent kernels above, which stream the matrices from
// the caches in every iteration: 4,040 us in the default schedule, 2,740 us in
// the best one.  Narrower shapes for narrow bands (12 entries, twice the
// waves) gained nothing: 693 us with the extra launches.
template <int B, int RPT, int W>
__global__ __launch_bounds__(B) __attribute__((amdgpu_waves_per_eu(RPT * W > 32 ? 2 : 4))) void k_batch_pcg_cls(
    const BatchDesc *__restrict__ desc, const double *__restrict__ ell_val, const short *__restrict__ ell_col,
    const double *__restrict__ dinv, const double *__restrict__ bvec, double *__restrict__ xout,
    int *__restrict__ iters_out, double *__restrict__ rel_out, uint8_t *__restrict__ status_out, double red_factor,
    int64_t max_iters_fixed, int iter_factor, int chk) {
    constexpr int G = W <= 12 ? 6 : 8;     // slots read from LDS at a time
    __shared__ double p_lds[B * RPT + 1];  // p, and a zero for the padding slots
    __shared__ double redA[8], redB[16], redC[16];
    const BatchDesc d = desc[blockIdx.x];
    const int n = d.n, w = d.w;
    double v[RPT][W];
    unsigned c[RPT][W / 2];
    double x[RPT], r[RPT], p[RPT], q[RPT], di[RPT];
    double rho = 0.0, bb = 0.0;
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        const int i = threadIdx.x + j * B;
        const bool own = i < n;
        const double *vp = ell_val + d.off + i;
        const short *cp = ell_col + d.off + i;
#pragma unroll
        for (int e = 0; e < W; e += 2) {
            double v0 = 0.0, v1 = 0.0;
            int c0 = -1, c1 = -1;
            if (own && e < w) {
                v0 = __builtin_nontemporal_load(vp + (int64_t)e * n);
                c0 = __builtin_nontemporal_load(cp + (int64_t)e * n);
            }
            if (own && e + 1 < w) {
                v1 = __builtin_nontemporal_load(vp + (int64_t)(e + 1) * n);
                c1 = __builtin_nontemporal_load(cp + (int64_t)(e + 1) * n);
            }
            v[j][e] = v0;
            v[j][e + 1] = v1;
            c[j][e / 2] = (unsigned)(c0 < 0 ? n : c0) * 8u | (unsigned)(c1 < 0 ? n : c1) * 8u << 16;
        }
        const double bi = own ? bvec[d.r0 + i] : 0.0;
        di[j] = own ? dinv[d.r0 + i] : 0.0;
        // x = 0, r = b, p = z = D^{-1} r
        x[j] = 0.0;
        r[j] = bi;
        p[j] = di[j] * bi;
        if (own) p_lds[i] = p[j];
        rho += r[j] * p[j];
        bb += bi * bi;
    }
    if (threadIdx.x == 0) p_lds[n] = 0.0;
    cls_sum2<B>(rho, bb, redC);
    const double nb = sqrt(bb), tol = red_factor * nb;
    bool by_top;
    const double top = norm2_bound(tol, by_top);  // sqrt(rr) <= tol without the root
    auto met = [&](double rr) { return by_top ? rr <= top : sqrt(rr) <= tol; };
    const int64_t maxit = max_iters_fixed > 0 ? max_iters_fixed : (int64_t)iter_factor * n;
    int stop = ST_RUN;
    int64_t k = 0;
    double rr = bb;
    if (bb == 0.0 || met(rr)) stop = ST_CONVERGED;
    while (stop == ST_RUN && k < maxit) {
        __syncthreads();  // p complete
        double eta = 0.0;
#pragma unroll
        for (int j = 0; j < RPT; ++j) q[j] = 0.0;
#pragma unroll
        for (int e = 0; e < W; e += G)
            if (e < w) {
                double pv[RPT][G];
#pragma unroll
                for (int j = 0; j < RPT; ++j)
#pragma unroll
                    for (int u = 0; u < G; ++u) {
                        if (e + u >= W) continue;
                        const unsigned o = (u & 1) ? c[j][(e + u) / 2] >> 16 : c[j][(e + u) / 2] & 0xffffu;
                        pv[j][u] = *(const double *)((const char *)p_lds + o);
                    }
#pragma unroll
                for (int u = 0; u < G; ++u)
#pragma unroll
                    for (int j = 0; j < RPT; ++j)
                        if (e + u < W) q[j] += v[j][e + u] * pv[j][u];
            }
#pragma unroll
        for (int j = 0; j < RPT; ++j) eta += p[j] * q[j];
        eta = cls_sum<B>(eta, redA);
        if (chk && !finite_d(eta)) { stop = ST_NONFINITE; break; }
        if (eta <= 0.0) { stop = ST_BREAKDOWN; break; }
        const double alpha = rho / eta;
        double rz = 0.0;
        rr = 0.0;
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            const bool own = (int)threadIdx.x + j * B < n;
            x[j] += alpha * p[j];
            r[j] = own ? r[j] - alpha * q[j] : 0.0;  // lanes past the last row stay out of the sums whatever alpha is
            q[j] = di[j] * r[j];                     // z
            rz += r[j] * q[j];
            rr += r[j] * r[j];
        }
        cls_sum2<B>(rz, rr, redB);
        ++k;
        if (chk && !finite_d(rr)) { stop = ST_NONFINITE; break; }
        if (met(rr)) { stop = ST_CONVERGED; break; }
        if (chk && !finite_d(rz)) { stop = ST_NONFINITE; break; }
        if (rz == 0.0) { stop = ST_BREAKDOWN; break; }
        const double beta = rz / rho;
        rho = rz;
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            const int i = threadIdx.x + j * B;
            p[j] = q[j] + beta * p[j];
            if (i < n) p_lds[i] = p[j];
        }
    }
    if (stop == ST_RUN) stop = ST_MAX_ITERS;
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        const int i = threadIdx.x + j * B;
        if (i < n) xout[d.r0 + i] = x[j];
    }
    if (threadIdx.x == 0) {
        iters_out[d.sys] = (int)k;
        rel_out[d.sys] = nb > 0.0 ? sqrt(rr) / nb : 0.0;
        status_out[d.sys] = (uint8_t)stop;
    }
}

// One workgroup per system: checks 0 <= col < n_s for every stored entry
// (lowest bad row into *bad) and, when ev is not null, writes the system's
// slot-major ELL copy (padding: value 0, column -1).
__global__ void k_batch_to_ell(const int *__restrict__ sys_ptr, const int *__restrict__ rp,
                               const int *__restrict__ col, const double *__restrict__ val,
                               const int64_t *__restrict__ ell_off, const int *__restrict__ ell_w,
                               double *__restrict__ ev, short *__restrict__ ec, int *__restrict__ bad) {
    const int s = blockIdx.x;
    const int r0 = sys_ptr[s], n = sys_ptr[s + 1] - r0;
    const int w = ev ? ell_w[s] : 0;
    const int64_t off = ev ? ell_off[s] : 0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const int e0 = rp[r0 + i], len = rp[r0 + i + 1] - e0;
        bool ok = true;
        for (int e = 0; e < len; ++e) {
            const int c = col[e0 + e];
            if (c < 0 || c >= n) ok = false;
        }
        if (!ok) atomicMin(bad, r0 + i);
        if (ev)
            for (int e = 0; e < w; ++e) {
                const bool in = e < len;
                ev[off + (int64_t)e * n + i] = in ? val[e0 + e] : 0.0;
                ec[off + (int64_t)e * n + i] = in ? (short)col[e0 + e] : (short)-1;
            }
    }
}

// The rows of a single-workgroup system, thread t owning rows t + j*B (j < RPT):
// their (at most W) entries in registers, the vector they are multiplied with in
// LDS (byte offsets; n <= 7680, so two fit a register, PACK).  Slot 0 holds the
// diagonal where the row stores one: its factor is the thread's own element, in
// a register, not an LDS read.
template <int B, int RPT, int W, bool PACK>
struct SmallRows {
    static constexpr int NC = PACK ? W / 2 : W - 1;
    double v[RPT][W];
    unsigned c[RPT][NC], c0[(RPT + 1) / 2];
    bool any0;  // a row of this wave has another entry in slot 0

    __device__ __forceinline__ void load(int n, const int *__restrict__ rp, const int *__restrict__ col,
                                         const double *__restrict__ val) {
        bool other = false;
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            const int i = (int)threadIdx.x + j * B;
            const bool own = i < n;
            const int e0 = own ? rp[i] : 0, e1 = own ? rp[i + 1] : 0;
            // padding points at the thread's own row (value 0): SPD systems
            // store their diagonal, so padding adds no new dependency
            const unsigned self = 8u * (unsigned)(own ? i : 0);
            int d = 0;
#pragma unroll
            for (int e = W - 1; e > 0; --e)
                if (e0 + e < e1 && col[e0 + e] == i) d = e;
            if (e0 < e1 && col[e0] == i) d = 0;
            unsigned t = self;
#pragma unroll
            for (int e = 0; e < W; ++e) {  // entry d to slot 0, the others in their order
                const int k = e0 + (e == 0 ? d : (e <= d ? e - 1 : e));
                const unsigned o = k < e1 ? 8u * (unsigned)col[k] : self;
                v[j][e] = k < e1 ? val[k] : 0.0;
                if (e == 0) t = o;
                else if constexpr (!PACK) c[j][e - 1] = o;
                else c[j][(e - 1) / 2] = (e - 1) & 1 ? c[j][(e - 1) / 2] | o << 16 : o;
            }
            c0[j / 2] = j & 1 ? c0[j / 2] | t << 16 : t;
            other |= t != self;
        }
        any0 = __any(other);
    }
    // q = A u for the thread's rows; own: the thread's elements of u, which
    // also stands in LDS
    __device__ __forceinline__ void product(const double (&own)[RPT], const double *u, double (&q)[RPT]) {
        const char *lds = (const char *)u;
#pragma unroll
        for (int j = 0; j < RPT; ++j) q[j] = v[j][0] * own[j];
        if (any0) {
#pragma unroll
            for (int j = 0; j < RPT; ++j)
                q[j] = v[j][0] * *(const double *)(lds + (j & 1 ? c0[j / 2] >> 16 : c0[j / 2] & 0xffffu));
        }
#pragma unroll
        for (int j = 0; j < RPT; ++j)
#pragma unroll
            for (int e = 0; e < W - 1; ++e) {
                unsigned o;
                if constexpr (PACK) {
                    // unpacked ahead of the iterations they would take twice the registers
                    if (!(e & 1)) asm volatile("" : "+v"(c[j][e / 2]));
                    o = e & 1 ? c[j][e / 2] >> 16 : c[j][e / 2] & 0xffffu;
                } else o = c[j][e];
                q[j] += v[j][e + 1] * *(const double *)(lds + o);
            }
    }
};

// Whole Jacobi-PCG of one small system in one workgroup: the rows, x, r, p and
// dinv in registers; p, which the product gathers, is mirrored in LDS.  An
// iteration is the product, two reductions and the updates, and touches no
// memory, but for what two shapes spill: 196 bytes a lane in <512, 2, 32>, 8 in
// <512, 8, 5>.
//
// Bound by one CU's iteration: vector instructions (61% of the cycles at 4096
// rows), the LDS reads of the product, three barriers, two reductions (lane
// moves, no LDS shuffles) and two quotients.  5-point systems, us a solve, with
// x and dinv in global memory and shuffles -> this: 64^2 734 -> 374 (1.85 an
// iteration), 32^2 303 -> 146, 16^2 162 -> 84.  1024 threads of four rows take
// 529 at 64^2 (twice the waves repeat the reductions), dots summed by halves
// 391.
template <int B, int RPT, int W>
__global__ __launch_bounds__(B) void k_small_pcg(int n, const int *__restrict__ rp,
                                                 const int *__restrict__ col,
                                                 const double *__restrict__ val,
                                                 const double *__restrict__ dinv,
                                                 const double *__restrict__ b,
                                                 double *__restrict__ xio, double red_factor,
                                                 int64_t maxit, int chk, void *__restrict__ out3) {
    __shared__ double p_lds[B * RPT];  // rows past n hold zeros that nobody reads
    constexpr int NW = B / kWave;
    __shared__ double redA[NW], redB[2 * NW], redC[2 * NW], redD[NW];
    const int tid = threadIdx.x;
    SmallRows<B, RPT, W, (W > 8)> A;
    double x[RPT], r[RPT], pr[RPT], dv[RPT], q[RPT];
    A.load(n, rp, col, val);
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        const int i = tid + j * B;
        const bool own = i < n;
        dv[j] = own ? dinv[i] : 0.0;
        x[j] = own ? xio[i] : 0.0;
        p_lds[i] = x[j];
    }
    __syncthreads();
    A.product(x, p_lds, q);
    double rho = 0.0, rr = 0.0, bb = 0.0;
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        const int i = tid + j * B;
        const double bi = i < n ? b[i] : 0.0;
        r[j] = bi - q[j];
        pr[j] = dv[j] * r[j];
        rho += r[j] * pr[j];
        rr += r[j] * r[j];
        bb += bi * bi;
    }
    __syncthreads();  // the initial guess in p_lds is consumed
#pragma unroll
    for (int j = 0; j < RPT; ++j) p_lds[tid + j * B] = pr[j];
    cls_sum2<B>(rho, rr, redC);
    bb = cls_sum<B>(bb, redD);
    const double nb = sqrt(bb), tol = red_factor * nb;
    bool by_top;
    const double top = norm2_bound(tol, by_top);
    auto met = [&](double s) { return by_top ? s <= top : sqrt(s) <= tol; };
    int stop = ST_RUN;
    int64_t k = 0;
    if (bb == 0.0) {
#pragma unroll
        for (int j = 0; j < RPT; ++j) x[j] = 0.0;
        stop = ST_CONVERGED;
    } else if (met(rr)) {
        stop = ST_CONVERGED;
    }
    while (stop == ST_RUN && k < maxit) {
        __syncthreads();  // p complete
        A.product(pr, p_lds, q);
        double eta = 0.0;
#pragma unroll
        for (int j = 0; j < RPT; ++j) eta += pr[j] * q[j];
        eta = cls_sum<B>(eta, redA);
        if (chk && !finite_d(eta)) { stop = ST_NONFINITE; break; }
        if (eta <= 0.0) { stop = ST_BREAKDOWN; break; }
        const double alpha = rho / eta;
        double rzn = 0.0;
        rr = 0.0;
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            x[j] += alpha * pr[j];
            r[j] -= alpha * q[j];
            q[j] = dv[j] * r[j];  // z
            rzn += r[j] * q[j];
            rr += r[j] * r[j];
        }
        cls_sum2<B>(rzn, rr, redB);
        ++k;
        if (chk && !finite_d(rr)) { stop = ST_NONFINITE; break; }
        if (met(rr)) { stop = ST_CONVERGED; break; }
        if (chk && !finite_d(rzn)) { stop = ST_NONFINITE; break; }
        if (rzn == 0.0) { stop = ST_BREAKDOWN; break; }
        const double beta = rzn / rho;
        rho = rzn;
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            pr[j] = q[j] + beta * pr[j];
            p_lds[tid + j * B] = pr[j];
        }
    }
    if (stop == ST_RUN) stop = ST_MAX_ITERS;
#pragma unroll
    for (int j = 0; j < RPT; ++j)
        if (tid + j * B < n) xio[tid + j * B] = x[j];
    if (tid == 0) {
        *(int32_t *)out3 = (int32_t)k;
        *(double *)((char *)out3 + 8) = nb > 0.0 ? sqrt(rr) / nb : 0.0;
        *((uint8_t *)out3 + 16) = (uint8_t)stop;
    }
}

// Whole Jacobi-BiCGSTAB of one small system in one workgroup, the steps
// and checks of the per-step solver in its order (right preconditioning,
// half-step exit x += alpha p_hat when ||s|| meets the criterion; rho of the
// next iteration is summed together with the residual norm).  The rows and r,
// r_hat, p, v, x and dinv stay in registers; the vector the product gathers
// (p_hat, then s_hat) is mirrored in LDS.  Between two writes of it lie the
// barriers of at least one reduction, as between two uses of a reduction's
// array.  <512, 8, 5> spills 136 bytes a lane.  out3: iterations (int32 at 0), relative residual
// (double at 8), status (byte 16), half step (byte 17).
template <int B, int RPT, int W>
__global__ __launch_bounds__(B) void k_small_bicgstab(int n, const int *__restrict__ rp,
                                                      const int *__restrict__ col,
                                                      const double *__restrict__ val,
                                                      const double *__restrict__ dinv,
                                                      const double *__restrict__ b,
                                                      double *__restrict__ xio, double red_factor,
                                                      int64_t maxit, int chk, void *__restrict__ out3) {
    __shared__ double pl[B * RPT];  // rows past n hold zeros that nobody reads
    constexpr int NW = B / kWave;
    __shared__ double redA[NW], redB[NW], redC[2 * NW], redD[2 * NW], redE[2 * NW], redF[NW];
    const int tid = threadIdx.x;
    SmallRows<B, RPT, W, (RPT * W > 32)> A;
    double r[RPT], rh[RPT], p[RPT], v[RPT], x[RPT], dv[RPT], h[RPT];
    A.load(n, rp, col, val);
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        const int i = tid + j * B;
        const bool own = i < n;
        dv[j] = own ? dinv[i] : 0.0;
        x[j] = own ? xio[i] : 0.0;
        pl[i] = x[j];
    }
    __syncthreads();
    A.product(x, pl, v);
    double rr = 0.0, bb = 0.0, rho = 0.0;
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        const int i = tid + j * B;
        const double bi = i < n ? b[i] : 0.0;
        r[j] = bi - v[j];
        rh[j] = r[j];
        p[j] = 0.0;
        v[j] = 0.0;
        rr += r[j] * r[j];
        bb += bi * bi;
    }
    rho = rr;  // r_hat = r
    cls_sum2<B>(rho, rr, redE);
    bb = cls_sum<B>(bb, redF);
    const double nb = sqrt(bb);
    const double tol = red_factor * nb;
    bool by_top;
    const double top = norm2_bound(tol, by_top);
    auto met = [&](double s) { return by_top ? s <= top : sqrt(s) <= tol; };
    int stop = ST_RUN, half = 0;
    int64_t k = 0;
    if (bb == 0.0) {
#pragma unroll
        for (int j = 0; j < RPT; ++j) x[j] = 0.0;
        stop = ST_CONVERGED;
    } else if (met(rr)) {
        stop = ST_CONVERGED;
    }
    double rho_old = 1.0, alpha = 1.0, omega = 1.0;
    while (stop == ST_RUN && k < maxit) {
        if (chk && !finite_d(rho)) { stop = ST_NONFINITE; break; }
        if (rho == 0.0) { stop = ST_BREAKDOWN; break; }
        const double beta = (rho / rho_old) * (alpha / omega);
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            p[j] = r[j] + beta * (p[j] - omega * v[j]);
            h[j] = dv[j] * p[j];
            pl[tid + j * B] = h[j];
        }
        __syncthreads();
        A.product(h, pl, v);
        double rv = 0.0;
#pragma unroll
        for (int j = 0; j < RPT; ++j) rv += rh[j] * v[j];
        rv = cls_sum<B>(rv, redA);
        if (chk && !finite_d(rv)) { stop = ST_NONFINITE; break; }
        if (rv == 0.0) { stop = ST_BREAKDOWN; break; }
        alpha = rho / rv;
        double ss = 0.0;
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            r[j] = r[j] - alpha * v[j];  // s
            ss += r[j] * r[j];
        }
        ++k;
        ss = cls_sum<B>(ss, redB);
        if (met(ss)) {
#pragma unroll
            for (int j = 0; j < RPT; ++j) x[j] += alpha * (dv[j] * p[j]);
            rr = ss;
            half = 1;
            stop = ST_CONVERGED;
            break;
        }
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            h[j] = dv[j] * r[j];
            pl[tid + j * B] = h[j];
        }
        __syncthreads();
        double tt = 0.0, ts = 0.0, t[RPT];
        A.product(h, pl, t);
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            tt += t[j] * t[j];
            ts += t[j] * r[j];
        }
        cls_sum2<B>(tt, ts, redC);
        if (chk && (!finite_d(tt) || !finite_d(ts))) { stop = ST_NONFINITE; break; }
        if (tt == 0.0) { stop = ST_BREAKDOWN; break; }
        omega = ts / tt;
        double rn = 0.0;
        rho_old = rho;
        rho = 0.0;
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            x[j] += alpha * (dv[j] * p[j]) + omega * (dv[j] * r[j]);
            r[j] = r[j] - omega * t[j];
            rn += r[j] * r[j];
            rho += rh[j] * r[j];
        }
        cls_sum2<B>(rn, rho, redD);
        rr = rn;
        if (chk && !finite_d(rn)) { stop = ST_NONFINITE; break; }
        if (met(rn)) { stop = ST_CONVERGED; break; }
        if (omega == 0.0) { stop = ST_BREAKDOWN; break; }
    }
    if (stop == ST_RUN) stop = ST_MAX_ITERS;
#pragma unroll
    for (int j = 0; j < RPT; ++j)
        if (tid + j * B < n) xio[tid + j * B] = x[j];
    if (tid == 0) {
        *(int32_t *)out3 = (int32_t)k;
        *(double *)((char *)out3 + 8) = nb > 0.0 ? sqrt(rr) / nb : 0.0;
        *((uint8_t *)out3 + 16) = (uint8_t)stop;
        *((uint8_t *)out3 + 17) = (uint8_t)half;
    }
}

__global__ void k_batch_jacobi(int64_t rows, const int *__restrict__ rows_sys_local_unused,
                               const int *__restrict__ rp, const int *__restrict__ col,
                               const double *__restrict__ val, const int *__restrict__ row_local,
                               double *__restrict__ dinv, int *__restrict__ bad) {
    (void)rows_sys_local_unused;
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= rows) return;
    const int li = row_local[i];
    double d = 0.0;
    bool found = false;
    for (int e = rp[i]; e < rp[i + 1]; ++e)
        if (col[e] == li) { d = val[e]; found = true; }
    if (found && d != 0.0) dinv[i] = 1.0 / d;
    else { dinv[i] = 0.0; atomicMin(bad, (int)i); }
}

__global__ void k_zero_u32(unsigned *p) { *p = 0u; }

// Fixed device scratch of mxl_batch_solve_noalloc: the work counter in the
// first 256 bytes, the spill region after it.  Each GPU that loads the
// library holds its own copy until the process ends.  Host code must not
// pass `noalloc_scratch` itself to a kernel (on the host it names a stand-in,
// not the device copy); it uses the address noalloc_scratch_init looked up.
constexpr size_t kNoAllocQueueBytes = 256;
__device__ __align__(256) unsigned char noalloc_scratch[kNoAllocScratchBytes];

namespace {
std::mutex g_noalloc_mu;
std::map<int, void *> g_noalloc_ptr;  // device -> address of that device's copy
}  // namespace

hipError_t noalloc_scratch_init(int device, void **out) {
    std::lock_guard<std::mutex> lk(g_noalloc_mu);
    auto it = g_noalloc_ptr.find(device);
    if (it != g_noalloc_ptr.end()) {
        *out = it->second;
        return hipSuccess;
    }
    void *ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(noalloc_scratch));
    if (e != hipSuccess || !ptr) {
        *out = nullptr;
        return e != hipSuccess ? e : hipErrorInvalidSymbol;
    }
    g_noalloc_ptr[device] = ptr;
    *out = ptr;
    return hipSuccess;
}

mxl_ctx *batch_ctx(const BatchImpl &B) { return B.ctx; }

}  // namespace mxl

using namespace mxl;

namespace {

size_t lds_bytes_for(int n) { return (size_t)4 * n * sizeof(double); }

// LDS bytes one workgroup of a schedule may use: all resident workgroups of
// a CU share its LDS.
int64_t lds_budget_for(const mxl_ctx *ctx, int wpc) {
    hipDeviceProp_t prop;
    size_t per_cu = 160 * 1024, per_wg = 64 * 1024;
    if (hipGetDeviceProperties(&prop, ctx->device) == hipSuccess) {
        if (prop.maxSharedMemoryPerMultiProcessor > 0) per_cu = prop.maxSharedMemoryPerMultiProcessor;
        if (prop.sharedMemPerBlock > 0) per_wg = prop.sharedMemPerBlock;
    }
    return (int64_t)std::min(per_wg, per_cu / (size_t)std::max(1, wpc)) - 2048;  // static LDS headroom
}

// Vector length of the CSR kernel's LDS vectors (x, r, p, q) for a schedule.
int lds_cap_for(const mxl_ctx *ctx, const BatchImpl &Bt, int wpc) {
    const int64_t budget = lds_budget_for(ctx, wpc);
    int cap = (int)(budget / (int64_t)(4 * sizeof(double)));
    return std::min(cap, Bt.max_n);
}

// The kernel a schedule runs: its format field, 0 choosing ELL when built.
bool use_ell(const BatchImpl &Bt, const mxl_tuning &t) { return t.format == 2 || (t.format == 0 && Bt.ell); }

// queue: the work counter (zeroed here by a kernel, not a memset, so the
// launch sequence can be captured); scr: the spill region, at least
// wgs_per_cu * num_cu * 5 * max_n doubles when any system spills, else NULL.
hipError_t launch_batch_on(const BatchImpl &Bt, const mxl_tuning &t, const mxl_criteria &c,
                           const double *b, double *x, int32_t *iters, double *rel, uint8_t *status,
                           int lds_cap, int64_t ell_budget, hipStream_t s, unsigned *queue, double *scr,
                           int use_x0 = 0, bool rest = false) {
    const int *order = rest ? (const int *)Bt.order_rest->p + (t.order ? Bt.nrest : 0)
                            : (const int *)(t.order ? Bt.order_big->p : Bt.order_input->p);
    const int64_t nsys = rest ? Bt.nrest : Bt.nsys;
    // beside the classes, no workgroup that would find nothing to do
    const int all = t.wgs_per_cu * Bt.ctx->num_cu, G = rest ? (int)std::min<int64_t>(all, nsys) : all;
    hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(1), 0, s, queue);
    const int chk = c.nonfinite_check;
    const double red = c.reduction;
    const int64_t mif = c.max_iters;
    if (use_ell(Bt, t)) {
        const size_t shm = (size_t)ell_budget;
        const int64_t stride = scr ? (int64_t)5 * Bt.max_n : 0;
#define MXL_BATCH_ELL_CASE(BB)                                                                       \
    case BB:                                                                                         \
        hipLaunchKernelGGL(k_batch_pcg_ell<BB>, dim3(G), dim3(BB), shm, s, nsys,                     \
                           (const int *)Bt.sys_ptr->p, (const int64_t *)Bt.ell_off->p,              \
                           (const int *)Bt.ell_w->p, (const double *)Bt.ell_val->p,                 \
                           (const short *)Bt.ell_col->p, (const double *)Bt.dinv->p, b, x, iters,   \
                           rel, status, order, queue, red, mif, 10, chk,                            \
                           ell_budget, scr, stride, use_x0);                                        \
        break;
        switch (t.wg_size) {
            MXL_BATCH_ELL_CASE(64) MXL_BATCH_ELL_CASE(128) MXL_BATCH_ELL_CASE(256) MXL_BATCH_ELL_CASE(512)
            MXL_BATCH_ELL_CASE(1024)
        default: return hipErrorInvalidValue;
        }
#undef MXL_BATCH_ELL_CASE
        return hipGetLastError();
    }
    const size_t shm = lds_bytes_for(lds_cap);
    const int64_t stride = scr ? (int64_t)4 * Bt.max_n : 0;
#define MXL_BATCH_CASE(BB)                                                                          \
    case BB:                                                                                        \
        hipLaunchKernelGGL(k_batch_pcg<BB>, dim3(G), dim3(BB), shm, s, nsys,                        \
                           (const int *)Bt.sys_ptr->p, (const int *)Bt.row_ptr->p,                 \
                           (const int *)Bt.col->p, (const double *)Bt.val->p,                      \
                           (const double *)Bt.dinv->p, b, x, iters, rel, status, order,            \
                           queue, red, mif, 10, chk, lds_cap, scr, stride, use_x0);                \
        break;
    switch (t.wg_size) {
        MXL_BATCH_CASE(64) MXL_BATCH_CASE(128) MXL_BATCH_CASE(256) MXL_BATCH_CASE(512) MXL_BATCH_CASE(1024)
    default: return hipErrorInvalidValue;
    }
#undef MXL_BATCH_CASE
    return hipGetLastError();
}

// The size-class schedule: a launch per class, largest first; the systems that no
// class holds (t: their schedule, as launch_batch_on) run beside them on a stream of
// the handle's own, between two events of the caller's stream: the largest
// systems take as long alone as among all, so that one after the other a few
// hundred systems of 32 to 3,000 rows took 2,047 us, side by side 1,293, all of them by
// the persistent kernel 1,517.
template <int K>
void launch_class(const BatchImpl &Bt, const mxl_criteria &c, const double *b, double *x, int32_t *iters,
                  double *rel, uint8_t *status, hipStream_t s) {
    const int64_t cnt = Bt.cls_begin[K + 1] - Bt.cls_begin[K];
    if (cnt > 0)
        hipLaunchKernelGGL((k_batch_pcg_cls<kClsN[K] / kClsR[K], kClsR[K], kClsW>), dim3((unsigned)cnt),
                           dim3(kClsN[K] / kClsR[K]), 0, s,
                           (const BatchDesc *)Bt.desc->p + Bt.cls_begin[K], (const double *)Bt.ell_val->p,
                           (const short *)Bt.ell_col->p, (const double *)Bt.dinv->p, b, x, iters, rel, status,
                           c.reduction, c.max_iters, 10, c.nonfinite_check);
}

hipError_t launch_classes(const BatchImpl &Bt, const mxl_tuning &t, const mxl_criteria &c, const double *b,
                          double *x, int32_t *iters, double *rel, uint8_t *status, int lds_cap, int64_t ell_budget,
                          hipStream_t s, unsigned *queue, double *scr) {
    hipError_t e = hipSuccess;
    const bool both = Bt.nrest > 0;
    if (both) {
        if ((e = hipEventRecord(Bt.fork, s)) != hipSuccess || (e = hipStreamWaitEvent(Bt.side, Bt.fork, 0)) != hipSuccess)
            return e;
        e = launch_batch_on(Bt, t, c, b, x, iters, rel, status, lds_cap, ell_budget, Bt.side, queue, scr, 0, true);
    }
    launch_class<4>(Bt, c, b, x, iters, rel, status, s);
    launch_class<3>(Bt, c, b, x, iters, rel, status, s);
    launch_class<2>(Bt, c, b, x, iters, rel, status, s);
    launch_class<1>(Bt, c, b, x, iters, rel, status, s);
    launch_class<0>(Bt, c, b, x, iters, rel, status, s);
    const hipError_t le = hipGetLastError();
    if (both) {  // whatever became of the launches, the caller's stream goes on after both
        const hipError_t r = hipEventRecord(Bt.join, Bt.side);
        const hipError_t w = r == hipSuccess ? hipStreamWaitEvent(s, Bt.join, 0) : r;
        if (e == hipSuccess) e = w;
    }
    return e == hipSuccess ? le : e;
}

// The handle's own queue counter and (lazily allocated) spill region.
hipError_t launch_batch(const BatchImpl &Bt, const mxl_tuning &t, const mxl_criteria &c,
                        const double *b, double *x, int32_t *iters, double *rel, uint8_t *status,
                        int lds_cap, int64_t ell_budget, hipStream_t s, int use_x0 = 0) {
    return launch_batch_on(Bt, t, c, b, x, iters, rel, status, lds_cap, ell_budget, s,
                           (unsigned *)Bt.queue->p, Bt.scratch ? (double *)Bt.scratch->p : nullptr,
                           use_x0);
}

}  // namespace

extern "C" mxl_status mxl_batch_csr_create(mxl_ctx *ctx, int64_t nsys, const int32_t *sys_ptr_host,
                                           const int32_t *sys_ptr, const int32_t *row_ptr,
                                           const int32_t *col, const double *val, int flags,
                                           mxl_op **out) try {
    (void)flags;
    if (!ctx || !out || !sys_ptr_host || nsys <= 0 || !sys_ptr || !row_ptr || !col || !val)
        return set_error(MXL_ERR_INVALID_ARG, "batch: NULL argument or nsys <= 0");
    *out = nullptr;
    auto Bt = std::make_shared<BatchImpl>();
    Bt->ctx = ctx;
    Bt->nsys = nsys;
    Bt->sys_ptr_h.assign(sys_ptr_host, sys_ptr_host + nsys + 1);
    if (Bt->sys_ptr_h[0] != 0) return set_error(MXL_ERR_INVALID_MATRIX, "sys_ptr[0] != 0");
    int max_n = 0;
    for (int64_t s = 0; s < nsys; ++s) {
        int n = Bt->sys_ptr_h[s + 1] - Bt->sys_ptr_h[s];
        if (n <= 0) return set_error(MXL_ERR_INVALID_MATRIX, "every system needs at least one row");
        max_n = std::max(max_n, n);
    }
    Bt->max_n = max_n;
    Bt->rows = Bt->sys_ptr_h[nsys];
    hipStream_t s = ctx->stream;
    int32_t nnz_h = 0;
    if (hipMemcpyAsync(&nnz_h, row_ptr + Bt->rows, 4, hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return set_error(MXL_ERR_INVALID_ARG, "row_ptr is not readable device memory");
    Bt->nnz = nnz_h;
    mxl_status st;
    if ((st = check_device_ptr(ctx, sys_ptr, (nsys + 1) * 4, "sys_ptr")) != MXL_OK) return st;
    if ((st = check_device_ptr(ctx, row_ptr, (Bt->rows + 1) * 4, "row_ptr")) != MXL_OK) return st;
    if ((st = check_device_ptr(ctx, col, Bt->nnz * 4, "col")) != MXL_OK) return st;
    if ((st = check_device_ptr(ctx, val, Bt->nnz * 8, "val")) != MXL_OK) return st;
    auto borrow = [](const void *p, size_t b) {
        auto d = std::make_shared<DevBuf>();
        d->p = const_cast<void *>(p);
        d->bytes = b;
        return d;
    };
    Bt->sys_ptr = borrow(sys_ptr, (nsys + 1) * 4);
    Bt->row_ptr = borrow(row_ptr, (Bt->rows + 1) * 4);
    Bt->col = borrow(col, Bt->nnz * 4);
    Bt->val = borrow(val, Bt->nnz * 8);
    auto alloc = [](size_t bytes) -> BufPtr {
        auto d = std::make_shared<DevBuf>();
        if (hipMalloc(&d->p, bytes ? bytes : 16) != hipSuccess) return nullptr;
        d->bytes = bytes;
        d->owned = true;
        return d;
    };
    Bt->dinv = alloc(Bt->rows * 8);
    Bt->order_input = alloc(nsys * 4);
    Bt->order_big = alloc(nsys * 4);
    Bt->queue = alloc(64);
    auto rowloc = alloc(Bt->rows * 4);
    auto bad = alloc(4);
    if (!Bt->dinv || !Bt->order_input || !Bt->order_big || !Bt->queue || !rowloc || !bad)
        return set_error(MXL_ERR_OUT_OF_MEMORY, "batch workspace");
    std::vector<int32_t> ord(nsys), loc(Bt->rows);
    std::iota(ord.begin(), ord.end(), 0);
    if (hipMemcpyAsync(Bt->order_input->p, ord.data(), nsys * 4, hipMemcpyHostToDevice, s) != hipSuccess)
        return set_error(MXL_ERR_DEVICE, "upload order");
    std::vector<int32_t> big(ord);
    std::stable_sort(big.begin(), big.end(), [&](int a, int b) {
        return Bt->sys_ptr_h[a + 1] - Bt->sys_ptr_h[a] > Bt->sys_ptr_h[b + 1] - Bt->sys_ptr_h[b];
    });
    for (int64_t sy = 0; sy < nsys; ++sy)
        for (int32_t r = Bt->sys_ptr_h[sy]; r < Bt->sys_ptr_h[sy + 1]; ++r) loc[r] = r - Bt->sys_ptr_h[sy];
    int init = INT_MAX;
    if (hipMemcpyAsync(Bt->order_big->p, big.data(), nsys * 4, hipMemcpyHostToDevice, s) != hipSuccess ||
        hipMemcpyAsync(rowloc->p, loc.data(), Bt->rows * 4, hipMemcpyHostToDevice, s) != hipSuccess ||
        hipMemcpyAsync(bad->p, &init, 4, hipMemcpyHostToDevice, s) != hipSuccess)
        return set_error(MXL_ERR_DEVICE, "upload batch tables");
    hipLaunchKernelGGL(k_batch_jacobi, dim3((unsigned)((Bt->rows + 255) / 256)), dim3(256), 0, s, Bt->rows,
                       nullptr, (const int *)row_ptr, col, val, (const int *)rowloc->p,
                       (double *)Bt->dinv->p, (int *)bad->p);
    int badh = INT_MAX;
    if (hipMemcpyAsync(&badh, bad->p, 4, hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return set_error(MXL_ERR_DEVICE, "batch jacobi");
    if (badh != INT_MAX)
        return set_error(MXL_ERR_ZERO_DIAG, "row " + std::to_string(badh) + " has a missing or zero diagonal");
    // Row lengths on the host: canonical row_ptr, and the per-system ELL
    // layout when it stays compact (<= 1.5 x the stored entries) and local
    // columns fit int16.
    std::vector<int32_t> rp_h((size_t)Bt->rows + 1);
    if (hipMemcpyAsync(rp_h.data(), row_ptr, ((size_t)Bt->rows + 1) * 4, hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return set_error(MXL_ERR_DEVICE, "read row_ptr");
    if (rp_h[0] != 0) return set_error(MXL_ERR_INVALID_MATRIX, "row_ptr[0] != 0");
    for (int64_t r = 0; r < Bt->rows; ++r)
        if (rp_h[r + 1] < rp_h[r]) return set_error(MXL_ERR_INVALID_MATRIX, "row_ptr decreases at row " + std::to_string(r));
    std::vector<int32_t> w_h(nsys);
    std::vector<int64_t> off_h(nsys);
    int64_t slots = 0;
    int w_max = 0;
    for (int64_t sy = 0; sy < nsys; ++sy) {
        int w = 0;
        for (int32_t r = Bt->sys_ptr_h[sy]; r < Bt->sys_ptr_h[sy + 1]; ++r) w = std::max(w, rp_h[r + 1] - rp_h[r]);
        w_h[sy] = w;
        w_max = std::max(w_max, w);
        off_h[sy] = slots;
        slots += ((int64_t)w * (Bt->sys_ptr_h[sy + 1] - Bt->sys_ptr_h[sy]) + 1) / 2 * 2;
    }
    const bool ell = max_n <= 32767 && (double)slots <= 1.5 * (double)Bt->nnz + 64.0 * (double)nsys;
    if (ell) {
        Bt->ell_val = alloc((size_t)slots * 8);
        Bt->ell_col = alloc((size_t)slots * 2);
        Bt->ell_off = alloc((size_t)nsys * 8);
        Bt->ell_w = alloc((size_t)nsys * 4);
        if (!Bt->ell_val || !Bt->ell_col || !Bt->ell_off || !Bt->ell_w)
            return set_error(MXL_ERR_OUT_OF_MEMORY, "batch ELL copy");
        if (hipMemcpyAsync(Bt->ell_off->p, off_h.data(), (size_t)nsys * 8, hipMemcpyHostToDevice, s) != hipSuccess ||
            hipMemcpyAsync(Bt->ell_w->p, w_h.data(), (size_t)nsys * 4, hipMemcpyHostToDevice, s) != hipSuccess)
            return set_error(MXL_ERR_DEVICE, "upload ELL tables");
        Bt->ell = true;
        Bt->w_max = w_max;
        Bt->ell_slots = slots;
        // size classes, each largest first (big is sorted by size); the rest
        // in the same order
        std::vector<BatchDesc> de;
        std::vector<int32_t> rest;
        de.reserve((size_t)nsys);
        auto cls_of = [&](int sy) {
            const int n = Bt->sys_ptr_h[sy + 1] - Bt->sys_ptr_h[sy];
            int k = 0;
            while (k < 5 && n > kClsN[k]) ++k;
            return w_h[sy] <= kClsW ? k : 5;
        };
        for (int k = 0; k <= 5; ++k) {
            Bt->cls_begin[k] = (int64_t)de.size();
            for (int32_t sy : big) {
                if (cls_of(sy) != k) continue;
                if (k == 5) rest.push_back(sy);
                else de.push_back({sy, Bt->sys_ptr_h[sy], Bt->sys_ptr_h[sy + 1] - Bt->sys_ptr_h[sy], w_h[sy], off_h[sy], 0});
            }
        }
        Bt->nrest = (int64_t)rest.size();
        std::vector<int32_t> by_input(rest);
        std::sort(by_input.begin(), by_input.end());
        rest.insert(rest.begin(), by_input.begin(), by_input.end());
        if (Bt->nrest > 0 && !de.empty() &&
            (hipStreamCreateWithFlags(&Bt->side, hipStreamNonBlocking) != hipSuccess ||
             hipEventCreateWithFlags(&Bt->fork, hipEventDisableTiming) != hipSuccess ||
             hipEventCreateWithFlags(&Bt->join, hipEventDisableTiming) != hipSuccess))
            return set_error(MXL_ERR_DEVICE, "batch side stream");
        // As long as every system can have a CU to itself, the largest decides, and the
        // launches beside it only cost: 20 systems of 32 to 3,000 rows 742 us by classes and
        // 702 without, 100 systems 1,142 either way, 300 1,293 against 1,510.
        Bt->cls_best = Bt->nrest == 0 || nsys > ctx->num_cu;
        Bt->desc = alloc(de.size() * sizeof(BatchDesc));
        Bt->order_rest = alloc(rest.size() * 4);
        if (!Bt->desc || !Bt->order_rest) return set_error(MXL_ERR_OUT_OF_MEMORY, "batch size classes");
        if ((!de.empty() && hipMemcpyAsync(Bt->desc->p, de.data(), de.size() * sizeof(BatchDesc), hipMemcpyHostToDevice,
                                           s) != hipSuccess) ||
            (!rest.empty() && hipMemcpyAsync(Bt->order_rest->p, rest.data(), rest.size() * 4, hipMemcpyHostToDevice,
                                             s) != hipSuccess) ||
            hipStreamSynchronize(s) != hipSuccess)  // the host lists end here
            return set_error(MXL_ERR_DEVICE, "upload size classes");
    }
    badh = INT_MAX;
    if (hipMemcpyAsync(bad->p, &badh, 4, hipMemcpyHostToDevice, s) != hipSuccess)
        return set_error(MXL_ERR_DEVICE, "upload flag");
    hipLaunchKernelGGL(k_batch_to_ell, dim3((unsigned)nsys), dim3(256), 0, s, sys_ptr, row_ptr, col, val,
                       ell ? (const int64_t *)Bt->ell_off->p : nullptr, ell ? (const int *)Bt->ell_w->p : nullptr,
                       ell ? (double *)Bt->ell_val->p : nullptr, ell ? (short *)Bt->ell_col->p : nullptr,
                       (int *)bad->p);
    if (hipMemcpyAsync(&badh, bad->p, 4, hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return set_error(MXL_ERR_DEVICE, "batch column check");
    if (badh != INT_MAX)
        return set_error(MXL_ERR_INVALID_MATRIX, "row " + std::to_string(badh) + " has a column outside its system");
    auto *op = new mxl_op;
    op->kind = MXL_OP_BATCH;
    op->bat = Bt;
    *out = op;
    return MXL_OK;
} catch (...) {
    return mxl::abi_exception(__func__);
}

static const BatchImpl *batch_of(const mxl_op *op) {
    return op && op->kind == MXL_OP_BATCH ? op->bat.get() : nullptr;
}

static mxl_status batch_args(const BatchImpl &Bt, const double *b, double *x, const int32_t *iters,
                             const double *rel, const uint8_t *status) {
    mxl_status st;
    const mxl_ctx *c = Bt.ctx;
    if ((st = check_device_ptr(c, b, Bt.rows * 8, "b")) != MXL_OK) return st;
    if ((st = check_device_ptr(c, x, Bt.rows * 8, "x")) != MXL_OK) return st;
    if ((st = check_device_ptr(c, iters, Bt.nsys * 4, "iters")) != MXL_OK) return st;
    if ((st = check_device_ptr(c, rel, Bt.nsys * 8, "rel_res")) != MXL_OK) return st;
    if ((st = check_device_ptr(c, status, Bt.nsys, "status")) != MXL_OK) return st;
    if ((const void *)b == (const void *)x) return set_error(MXL_ERR_INVALID_ARG, "b and x alias");
    return MXL_OK;
}

// Dynamic LDS above 64 KB needs the kernel's attribute raised first.
#define MXL_ALLOW_LDS(KERN, WG, SHM)                                                                    \
    [&]() -> hipError_t {                                                                               \
        if ((SHM) <= 64 * 1024) return hipSuccess;                                                      \
        const int v_ = (int)(SHM);                                                                      \
        switch (WG) {                                                                                   \
        case 64: return hipFuncSetAttribute((const void *)KERN<64>, hipFuncAttributeMaxDynamicSharedMemorySize, v_);   \
        case 128: return hipFuncSetAttribute((const void *)KERN<128>, hipFuncAttributeMaxDynamicSharedMemorySize, v_); \
        case 256: return hipFuncSetAttribute((const void *)KERN<256>, hipFuncAttributeMaxDynamicSharedMemorySize, v_); \
        case 512: return hipFuncSetAttribute((const void *)KERN<512>, hipFuncAttributeMaxDynamicSharedMemorySize, v_); \
        default: return hipFuncSetAttribute((const void *)KERN<1024>, hipFuncAttributeMaxDynamicSharedMemorySize, v_); \
        }                                                                                               \
    }()

// What a schedule needs: its kernel, that kernel's LDS, and the spill region
// (doubles) when the largest system does not fit in LDS.
struct SchedPlan {
    bool ell = false;
    int cap = 0;
    int64_t ell_budget = 0;
    int64_t spill_elems = 0;
};

static mxl_status plan_schedule(const BatchImpl &Bt, const mxl_tuning &t, SchedPlan &p) {
    if (t.wg_size != 64 && t.wg_size != 128 && t.wg_size != 256 && t.wg_size != 512 && t.wg_size != 1024)
        return set_error(MXL_ERR_INVALID_ARG, "wg_size must be 64, 128, 256, 512 or 1024");
    if (t.wgs_per_cu < 1 || t.wgs_per_cu > 32 || (t.order != 0 && t.order != 1))
        return set_error(MXL_ERR_INVALID_ARG, "wgs_per_cu in 1..32, order 0 or 1");
    if (t.format < 0 || t.format > 2) return set_error(MXL_ERR_INVALID_ARG, "format must be 0, 1 or 2");
    if (t.format == 2 && !Bt.ell)
        return set_error(MXL_ERR_NOT_IMPLEMENTED, "this batch has no compact ELL copy (format 2)");
    p.ell = use_ell(Bt, t);
    p.cap = lds_cap_for(Bt.ctx, Bt, t.wgs_per_cu);
    // the ELL kernel's LDS: at most what the largest system can use
    p.ell_budget = std::min(lds_budget_for(Bt.ctx, t.wgs_per_cu),
                            (int64_t)Bt.max_n * (40 + 10 * (int64_t)Bt.w_max));
    if (p.cap < 1 || p.ell_budget < 40) return set_error(MXL_ERR_INVALID_ARG, "schedule leaves no LDS per workgroup");
    const bool spill = p.ell ? (int64_t)40 * Bt.max_n > p.ell_budget : p.cap < Bt.max_n;
    // systems above the LDS capacity run from a global scratch slice per workgroup
    p.spill_elems = spill ? (int64_t)t.wgs_per_cu * Bt.ctx->num_cu * 5 * Bt.max_n : 0;
    return MXL_OK;
}

static mxl_status allow_lds(const SchedPlan &p, const mxl_tuning &t) {
    hipError_t e = p.ell ? MXL_ALLOW_LDS(k_batch_pcg_ell, t.wg_size, (size_t)p.ell_budget)
                         : MXL_ALLOW_LDS(k_batch_pcg, t.wg_size, lds_bytes_for(p.cap));
    if (e != hipSuccess) return set_error(MXL_ERR_DEVICE, std::string("LDS attribute: ") + hipGetErrorString(e));
    return MXL_OK;
}

static mxl_status run_schedule(BatchImpl &Bt, const mxl_tuning &t, const mxl_criteria &c,
                               const double *b, double *x, int32_t *iters, double *rel,
                               uint8_t *status, bool classes = false) {
    SchedPlan p;
    mxl_status st;
    if ((st = plan_schedule(Bt, t, p)) != MXL_OK) return st;
    if (classes && Bt.nrest == 0) p.spill_elems = 0;
    if (p.spill_elems > 0 && Bt.scratch_elems < p.spill_elems) {
        auto d = std::make_shared<DevBuf>();
        if (hipMalloc(&d->p, p.spill_elems * 8) != hipSuccess)
            return set_error(MXL_ERR_OUT_OF_MEMORY, "batch scratch");
        d->bytes = p.spill_elems * 8;
        d->owned = true;
        Bt.scratch = d;
        Bt.scratch_elems = p.spill_elems;
    }
    if ((st = allow_lds(p, t)) != MXL_OK) return st;
    hipError_t e = classes ? launch_classes(Bt, t, c, b, x, iters, rel, status, p.cap, p.ell_budget, Bt.ctx->stream,
                                            (unsigned *)Bt.queue->p, Bt.scratch ? (double *)Bt.scratch->p : nullptr)
                           : launch_batch(Bt, t, c, b, x, iters, rel, status, p.cap, p.ell_budget, Bt.ctx->stream);
    if (e != hipSuccess) return set_error(MXL_ERR_DEVICE, std::string("batched launch: ") + hipGetErrorString(e));
    return MXL_OK;
}

// Whether calls without a schedule run by size class.
static bool by_class(const BatchImpl &Bt) {
    return Bt.ell && Bt.cls_best && Bt.cls_begin[5] > 0;
}

static mxl_tuning default_tuning() {
    mxl_tuning t;
    t.wg_size = 256;
    t.wgs_per_cu = 2;
    t.order = 0;
    t.format = 0;
    return t;
}

extern "C" mxl_status mxl_batch_solve(const mxl_op *Bop, const mxl_criteria *crit, const mxl_tuning *tuning,
                                      const double *b, double *x, int32_t *iters, double *rel_res,
                                      uint8_t *status) try {
    BatchImpl *Bt = const_cast<BatchImpl *>(batch_of(Bop));
    if (!Bt || !crit) return set_error(MXL_ERR_INVALID_ARG, "batch operator and criteria required");
    if (!(crit->reduction >= 0.0)) return set_error(MXL_ERR_INVALID_ARG, "reduction must be >= 0");
    mxl_status st;
    if ((st = batch_args(*Bt, b, x, iters, rel_res, status)) != MXL_OK) return st;
    mxl_tuning t = tuning ? *tuning : (Bt->tuned ? Bt->best : default_tuning());
    if ((st = run_schedule(*Bt, t, *crit, b, x, iters, rel_res, status, !tuning && by_class(*Bt))) != MXL_OK) return st;
    if (hipStreamSynchronize(Bt->ctx->stream) != hipSuccess)
        return set_error(MXL_ERR_DEVICE, "batched solve");
    return MXL_OK;
} catch (...) {
    return mxl::abi_exception(__func__);
}

extern "C" mxl_status mxl_batch_solve_noalloc(const mxl_op *Bop, const mxl_criteria *crit,
                                              const mxl_tuning *tuning, const double *b, double *x,
                                              int32_t *iters, double *rel_res, uint8_t *status) try {
    BatchImpl *Bt = const_cast<BatchImpl *>(batch_of(Bop));
    if (!Bt || !crit) return set_error(MXL_ERR_INVALID_ARG, "batch operator and criteria required");
    if (!(crit->reduction >= 0.0)) return set_error(MXL_ERR_INVALID_ARG, "reduction must be >= 0");
    mxl_status st;
    if ((st = batch_args(*Bt, b, x, iters, rel_res, status)) != MXL_OK) return st;
    const mxl_tuning t = tuning ? *tuning : (Bt->tuned ? Bt->best : default_tuning());
    const bool classes = !tuning && by_class(*Bt);
    SchedPlan p;
    if ((st = plan_schedule(*Bt, t, p)) != MXL_OK) return st;
    if (classes && Bt->nrest == 0) p.spill_elems = 0;
    const size_t need = kNoAllocQueueBytes + (size_t)p.spill_elems * 8;
    if (need > kNoAllocScratchBytes)
        return set_error(MXL_ERR_INVALID_ARG,
                         "schedule needs " + std::to_string(need) + " bytes of scratch; the static limit is " +
                             std::to_string(kNoAllocScratchBytes) + " (fewer workgroups per CU spill less)");
    char *base = (char *)Bt->ctx->noalloc_scratch;
    if (!base) return set_error(MXL_ERR_DEVICE, "static scratch address not available on this device");
    if ((st = allow_lds(p, t)) != MXL_OK) return st;
    double *spill = p.spill_elems > 0 ? (double *)(base + kNoAllocQueueBytes) : nullptr;
    hipError_t e = classes ? launch_classes(*Bt, t, *crit, b, x, iters, rel_res, status, p.cap, p.ell_budget,
                                            Bt->ctx->stream, (unsigned *)base, spill)
                           : launch_batch_on(*Bt, t, *crit, b, x, iters, rel_res, status, p.cap, p.ell_budget,
                                             Bt->ctx->stream, (unsigned *)base, spill);
    if (e != hipSuccess) return set_error(MXL_ERR_DEVICE, std::string("batched launch: ") + hipGetErrorString(e));
    return MXL_OK;
} catch (...) {
    return mxl::abi_exception(__func__);
}

extern "C" mxl_status mxl_batch_autotune(const mxl_op *Bop, const mxl_criteria *crit, const double *b,
                                         double *x_scratch, int reps, mxl_tuning *best_out,
                                         double *best_ms) try {
    BatchImpl *Bt = const_cast<BatchImpl *>(batch_of(Bop));
    if (!Bt || !crit || reps < 1) return set_error(MXL_ERR_INVALID_ARG, "batch operator, criteria, reps >= 1");
    mxl_status st;
    if ((st = check_device_ptr(Bt->ctx, b, Bt->rows * 8, "b")) != MXL_OK) return st;
    if ((st = check_device_ptr(Bt->ctx, x_scratch, Bt->rows * 8, "x_scratch")) != MXL_OK) return st;
    hipStream_t s = Bt->ctx->stream;
    void *it = nullptr, *rl = nullptr, *stt = nullptr;
    if (hipMalloc(&it, Bt->nsys * 4) != hipSuccess || hipMalloc(&rl, Bt->nsys * 8) != hipSuccess ||
        hipMalloc(&stt, Bt->nsys) != hipSuccess) {
        (void)hipFree(it); (void)hipFree(rl); (void)hipFree(stt);
        return set_error(MXL_ERR_OUT_OF_MEMORY, "autotune buffers");
    }
    hipEvent_t e0, e1;
    (void)hipEventCreate(&e0);
    (void)hipEventCreate(&e1);
    double best = 1e300, cls_ms = 1e300;
    mxl_tuning bt = default_tuning();
    st = MXL_OK;
    // one schedule, timed reps times after a run that warms the caches
    auto timed = [&](const mxl_tuning &t, bool classes) {
        std::vector<float> ts;
        for (int r = 0; r < reps + 1 && st == MXL_OK; ++r) {
            (void)hipEventRecord(e0, s);
            st = run_schedule(*Bt, t, *crit, b, x_scratch, (int32_t *)it, (double *)rl, (uint8_t *)stt, classes);
            (void)hipEventRecord(e1, s);
            (void)hipEventSynchronize(e1);
            float ms = 0.f;
            (void)hipEventElapsedTime(&ms, e0, e1);
            if (r > 0) ts.push_back(ms);
        }
        std::sort(ts.begin(), ts.end());
        return ts.empty() ? 1e300 : (double)ts[ts.size() / 2];
    };
    std::vector<int> fmts{1};
    if (Bt->ell) fmts.push_back(2);
    for (int fmt : fmts) {
    if (st != MXL_OK) break;
    for (int B : {64, 128, 256, 512}) {
        for (int wpc : {1, 2, 4, 8}) {
            if (B * wpc > 2048) continue;  // at most 32 waves per CU
            for (int ord : {0, 1}) {
                mxl_tuning t{B, wpc, ord, fmt};
                const double med = timed(t, false);
                if (st != MXL_OK) break;
                if (med < best) { best = med; bt = t; }
            }
            if (st != MXL_OK) break;
        }
        if (st != MXL_OK) break;
    }
    }
    // the size-class schedule, with the best of them for the systems no class holds
    if (st == MXL_OK && Bt->ell && Bt->cls_begin[5] > 0) cls_ms = timed(bt, true);
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    (void)hipFree(it); (void)hipFree(rl); (void)hipFree(stt);
    if (st != MXL_OK) return st;
    Bt->cls_best = cls_ms <= best;
    Bt->best = bt;
    Bt->tuned = true;
    if (best_out) *best_out = bt;
    if (best_ms) *best_ms = best;
    return MXL_OK;
} catch (...) {
    return mxl::abi_exception(__func__);
}

namespace mxl {

// A single system (a solver's matrix) viewed as a batch of one, for the
// one-launch CG path of small systems.
std::shared_ptr<BatchImpl> batch_from_matrix(const MatrixImpl &A, const void *dinv) {
    auto Bt = std::make_shared<BatchImpl>();
    Bt->ctx = A.ctx;
    Bt->nsys = 1;
    Bt->rows = A.nrows;
    Bt->nnz = A.nnz;
    Bt->sys_ptr_h = {0, (int32_t)A.nrows};
    Bt->max_n = (int)A.nrows;
    Bt->row_ptr = A.row_ptr;
    Bt->col = A.col;
    Bt->val = A.val;
    auto alloc = [](size_t bytes) -> BufPtr {
        auto d = std::make_shared<DevBuf>();
        if (hipMalloc(&d->p, bytes ? bytes : 16) != hipSuccess) return nullptr;
        d->bytes = bytes;
        d->owned = true;
        return d;
    };
    Bt->sys_ptr = alloc(8);
    Bt->order_input = alloc(4);
    Bt->order_big = Bt->order_input;
    Bt->queue = alloc(64);
    Bt->scratch = nullptr;
    if (!Bt->sys_ptr || !Bt->order_input || !Bt->queue) return nullptr;
    if (dinv) {
        Bt->dinv = std::make_shared<DevBuf>();
        Bt->dinv->p = const_cast<void *>(dinv);
        Bt->dinv->bytes = A.nrows * 8;
    } else {
        Bt->dinv = alloc(A.nrows * 8);
        if (!Bt->dinv || launch_fill(MXL_F64, A.nrows, 1.0, Bt->dinv->p, A.ctx->stream) != hipSuccess) return nullptr;
    }
    int32_t sp[2] = {0, (int32_t)A.nrows}, z = 0;
    if (hipMemcpyAsync(Bt->sys_ptr->p, sp, 8, hipMemcpyHostToDevice, A.ctx->stream) != hipSuccess ||
        hipMemcpyAsync(Bt->order_input->p, &z, 4, hipMemcpyHostToDevice, A.ctx->stream) != hipSuccess ||
        hipStreamSynchronize(A.ctx->stream) != hipSuccess)
        return nullptr;
    return Bt;
}

// The whole CG of one system in one workgroup (x holds the initial guess).
// Register-cached single-workgroup shapes: (threads, rows per thread,
// entries per row), by rising work an iteration.  The first that holds the
// system is used.
struct SmallShape {
    int B, RPT, W;
};
static const SmallShape kSmallShapes[] = {{64, 2, 8},  {256, 2, 8}, {512, 2, 5},  {512, 2, 8},
                                          {512, 4, 5}, {512, 4, 8}, {512, 2, 32}, {512, 8, 5}};

// Index of the first shape that holds n rows of at most maxlen entries (ns: none).
static int small_fit(const SmallShape *shapes, int ns, int n, int maxlen) {
    for (int k = 0; k < ns; ++k)
        if (n <= shapes[k].B * shapes[k].RPT && maxlen <= shapes[k].W) return k;
    return ns;
}

static hipError_t launch_small(const SmallShape &sh, int n, const BatchImpl &Bt, const mxl_criteria &c,
                               const double *b, double *x, void *out3) {
    hipStream_t s = Bt.ctx->stream;
#define MXL_SMALL(BB, RR, WW)                                                                        \
    if (sh.B == BB && sh.RPT == RR && sh.W == WW) {                                                  \
        hipLaunchKernelGGL((k_small_pcg<BB, RR, WW>), dim3(1), dim3(BB), 0, s, n,                    \
                           (const int *)Bt.row_ptr->p, (const int *)Bt.col->p,                       \
                           (const double *)Bt.val->p, (const double *)Bt.dinv->p, b, x,              \
                           c.reduction, c.max_iters, c.nonfinite_check, out3);                       \
        return hipGetLastError();                                                                    \
    }
    MXL_SMALL(64, 2, 8)
    MXL_SMALL(256, 2, 8)
    MXL_SMALL(512, 2, 5)
    MXL_SMALL(512, 2, 8)
    MXL_SMALL(512, 4, 5)
    MXL_SMALL(512, 4, 8)
    MXL_SMALL(512, 2, 32)
    MXL_SMALL(512, 8, 5)
#undef MXL_SMALL
    return hipErrorInvalidValue;
}

// The whole BiCGSTAB of one system in one workgroup, when a register shape
// holds it (returns false otherwise; the caller then runs the per-step
// solver).  x holds the initial guess.
static const SmallShape kSmallBiShapes[] = {{64, 2, 8}, {256, 2, 8}, {512, 2, 8}, {512, 4, 5}, {512, 8, 5}};

bool batch_single_bicgstab(BatchImpl &Bt, const mxl_criteria &c, const double *b, double *x, void *out3,
                           int64_t *iters, double *rel, int *stop, int *half, mxl_status *st) {
    *st = MXL_OK;
    const int n = (int)Bt.rows;
    constexpr int NS = (int)(sizeof(kSmallBiShapes) / sizeof(kSmallBiShapes[0]));
    if (Bt.small_bi_shape < 0) {
        std::vector<int32_t> rp(n + 1);
        if (hipMemcpyAsync(rp.data(), Bt.row_ptr->p, (n + 1) * 4, hipMemcpyDeviceToHost, Bt.ctx->stream) != hipSuccess ||
            hipStreamSynchronize(Bt.ctx->stream) != hipSuccess) {
            *st = set_error(MXL_ERR_DEVICE, "row pointer read");
            return true;
        }
        int maxlen = 0;
        for (int i = 0; i < n; ++i) maxlen = std::max(maxlen, rp[i + 1] - rp[i]);
        Bt.small_bi_shape = small_fit(kSmallBiShapes, NS, n, maxlen);
    }
    if (Bt.small_bi_shape >= NS) return false;
    const SmallShape &sh = kSmallBiShapes[Bt.small_bi_shape];
    hipStream_t s = Bt.ctx->stream;
#define MXL_SMALL_BI(BB, RR, WW)                                                                     \
    if (sh.B == BB && sh.RPT == RR && sh.W == WW)                                                    \
        hipLaunchKernelGGL((k_small_bicgstab<BB, RR, WW>), dim3(1), dim3(BB), 0, s, n,                \
                           (const int *)Bt.row_ptr->p, (const int *)Bt.col->p,                       \
                           (const double *)Bt.val->p, (const double *)Bt.dinv->p, b, x,              \
                           c.reduction, c.max_iters, c.nonfinite_check, out3);
    MXL_SMALL_BI(64, 2, 8)
    MXL_SMALL_BI(256, 2, 8)
    MXL_SMALL_BI(512, 2, 8)
    MXL_SMALL_BI(512, 4, 5)
    MXL_SMALL_BI(512, 8, 5)
#undef MXL_SMALL_BI
    hipError_t e = hipGetLastError();
    char h[24];
    if (e == hipSuccess) e = hipMemcpyAsync(h, out3, 24, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
        *st = set_error(MXL_ERR_DEVICE, std::string("small BiCGSTAB: ") + hipGetErrorString(e));
        return true;
    }
    int32_t it;
    memcpy(&it, h, 4);
    memcpy(rel, h + 8, 8);
    *iters = it;
    *stop = (uint8_t)h[16];
    *half = (uint8_t)h[17];
    return true;
}

static constexpr int kNumSmall = (int)(sizeof(kSmallShapes) / sizeof(kSmallShapes[0]));

// Whether a register shape holds the system (decided once: the longest row
// needs the row pointers).
bool batch_single_fits(BatchImpl &Bt, mxl_status *st) {
    *st = MXL_OK;
    const int n = (int)Bt.rows;
    if (Bt.small_shape < 0) {
        std::vector<int32_t> rp(n + 1);
        if (hipMemcpyAsync(rp.data(), Bt.row_ptr->p, (n + 1) * 4, hipMemcpyDeviceToHost, Bt.ctx->stream) != hipSuccess ||
            hipStreamSynchronize(Bt.ctx->stream) != hipSuccess) {
            *st = set_error(MXL_ERR_DEVICE, "row pointer read");
            return false;
        }
        int maxlen = 0;
        for (int i = 0; i < n; ++i) maxlen = std::max(maxlen, rp[i + 1] - rp[i]);
        Bt.small_shape = small_fit(kSmallShapes, kNumSmall, n, maxlen);
    }
    return Bt.small_shape < kNumSmall;
}

mxl_status batch_single_solve(BatchImpl &Bt, const mxl_criteria &c, const double *b, double *x,
                              void *out3, int64_t *iters, double *rel, int *stop) {
    const int n = (int)Bt.rows;
    mxl_status fit;
    const bool small = batch_single_fits(Bt, &fit);
    if (fit != MXL_OK) return fit;
    if (small) {
        hipError_t e = launch_small(kSmallShapes[Bt.small_shape], n, Bt, c, b, x, out3);
        if (e != hipSuccess) return set_error(MXL_ERR_DEVICE, std::string("small CG: ") + hipGetErrorString(e));
        char h[24];
        if (hipMemcpyAsync(h, out3, 24, hipMemcpyDeviceToHost, Bt.ctx->stream) != hipSuccess ||
            hipStreamSynchronize(Bt.ctx->stream) != hipSuccess)
            return set_error(MXL_ERR_DEVICE, "small CG read-back");
        int32_t it;
        memcpy(&it, h, 4);
        memcpy(rel, h + 8, 8);
        *iters = it;
        *stop = (uint8_t)h[16];
        return MXL_OK;
    }
    mxl_tuning t{1024, 1, 0, 1};
    const int cap = lds_cap_for(Bt.ctx, Bt, 1);
    if (cap < Bt.max_n && !Bt.scratch) {
        auto d = std::make_shared<DevBuf>();
        if (hipMalloc(&d->p, (size_t)Bt.ctx->num_cu * 4 * Bt.max_n * 8) != hipSuccess)
            return set_error(MXL_ERR_OUT_OF_MEMORY, "single-launch scratch");
        d->bytes = (size_t)Bt.ctx->num_cu * 4 * Bt.max_n * 8;
        d->owned = true;
        Bt.scratch = d;
        Bt.scratch_elems = (int64_t)Bt.ctx->num_cu * 4 * Bt.max_n;
    }
    const size_t shm = lds_bytes_for(cap);
    if (shm > 64 * 1024 &&
        hipFuncSetAttribute((const void *)k_batch_pcg<1024>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm) != hipSuccess)
        return set_error(MXL_ERR_DEVICE, "LDS attribute");
    int32_t *dit = (int32_t *)out3;
    double *drel = (double *)((char *)out3 + 8);
    uint8_t *dst = (uint8_t *)((char *)out3 + 16);
    hipError_t e = launch_batch(Bt, t, c, b, x, dit, drel, dst, cap, 0, Bt.ctx->stream, 1);
    if (e != hipSuccess) return set_error(MXL_ERR_DEVICE, std::string("single-launch CG: ") + hipGetErrorString(e));
    char h[24];
    if (hipMemcpyAsync(h, out3, 24, hipMemcpyDeviceToHost, Bt.ctx->stream) != hipSuccess ||
        hipStreamSynchronize(Bt.ctx->stream) != hipSuccess)
        return set_error(MXL_ERR_DEVICE, "single-launch read-back");
    int32_t it;
    memcpy(&it, h, 4);
    memcpy(rel, h + 8, 8);
    *iters = it;
    *stop = (uint8_t)h[16];
    return MXL_OK;
}

}  // namespace mxl
