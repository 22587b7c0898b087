// ilu.hip -- ILU-type preconditioner (Sec. 3.2): incomplete LU factors on
// A's sparsity pattern generated by ParILU, the fine-grained fixed-point
// method the paper cites, and applied by a lower and an upper triangular
// solve, exact (level-scheduled substitution) or iterative (Jacobi sweeps).
//
// Factors live in A's CSR pattern: the strictly lower entries are L (unit
// diagonal implied), the diagonal and upper entries U.  A ParILU sweep
// recomputes every entry (i, j) from the previous sweep's factors
//   s = a_ij - sum_{k < min(i,j)} l_ik u_kj,  l_ij = s / u_jj (i > j), u_ij = s
// one thread per entry, u_kj found by binary search in row k.  Sweeps are
// synchronous (double-buffered), so the factors after any number of sweeps
// are deterministic; with contraction off and the sums in ascending k they
// are the same numbers as a sequential evaluation.
#include <algorithm>
#include <climits>
#include <cstring>
#include <vector>

#include "device_common.hpp"
#include "ilu_levels.hpp"
#include "internal.hpp"

namespace mxl {

__device__ __forceinline__ int64_t row_find(const int *__restrict__ rp, const int *__restrict__ col, int64_t row,
                                            int c) {
    int64_t lo = rp[row], hi = (int64_t)rp[row + 1] - 1;
    while (lo <= hi) {
        const int64_t mid = lo + (hi - lo) / 2;
        const int v = col[mid];
        if (v == c) return mid;
        if (v < c) lo = mid + 1;
        else hi = mid - 1;
    }
    return -1;
}

// Diagonal position of every row; the first row whose diagonal is missing
// or zero goes to *bad.
__global__ void k_ilu_diag(int64_t n, const int *__restrict__ rp, const int *__restrict__ col,
                           const double *__restrict__ val, int *__restrict__ dpos, int *bad) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t p = row_find(rp, col, i, (int)i);
    dpos[i] = p < 0 ? rp[i] : (int)p;  // in bounds for what runs before the host has seen *bad
    if (p < 0 || val[p] == 0.0) atomicMin(bad, (int)(i < INT_MAX ? i : INT_MAX));
}

// Initial factors: l_ij = a_ij / a_jj, u_ij = a_ij.
__global__ void k_ilu_init(int64_t nnz, const int *__restrict__ row, const int *__restrict__ col,
                           const double *__restrict__ val, const int *__restrict__ dpos, double *__restrict__ lu) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= nnz) return;
    const int j = col[q];
    lu[q] = j < row[q] ? val[q] / val[dpos[j]] : val[q];
}

__global__ void k_parilu_sweep(int64_t nnz, const int *__restrict__ rp, const int *__restrict__ row,
                               const int *__restrict__ col, const double *__restrict__ val,
                               const int *__restrict__ dpos, const double *__restrict__ old,
                               double *__restrict__ lu) {
#pragma clang fp contract(off)
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= nnz) return;
    const int i = row[q], j = col[q];
    const int m = i < j ? i : j;
    double s = val[q];
    for (int64_t t = rp[i]; t < rp[i + 1]; ++t) {
        const int k = col[t];
        if (k >= m) break;
        const int64_t p = row_find(rp, col, k, j);
        if (p >= 0) s = s - old[t] * old[p];
    }
    lu[q] = i > j ? s / old[dpos[j]] : s;
}

// One row of each exact substitution.  The row's first kTrsBatch (column,
// factor) pairs are loaded together and its dependencies gathered together
// before any is used, so a row costs three round trips to memory (row
// bounds, entries, dependencies) instead of one per entry; the arithmetic
// is the sequential one, entry by entry in column order.
constexpr int kTrsBatch = 8;

__device__ __forceinline__ void trs_lower_row(int i, const int *__restrict__ rp, const int *__restrict__ col,
                                              const double *__restrict__ lu, const double *__restrict__ r,
                                              double *y) {
#pragma clang fp contract(off)
    const int q0 = rp[i], q1 = rp[i + 1];
    int c[kTrsBatch];
    double a[kTrsBatch], yv[kTrsBatch];
#pragma unroll
    for (int m = 0; m < kTrsBatch; ++m) {
        const int q = q0 + m;
        const bool in = q < q1;
        c[m] = in ? col[q] : INT_MAX;
        a[m] = in ? lu[q] : 0.0;
    }
#pragma unroll
    for (int m = 0; m < kTrsBatch; ++m) yv[m] = c[m] < i ? y[c[m]] : 0.0;
    double s = r[i];
    bool done = false;
#pragma unroll
    for (int m = 0; m < kTrsBatch; ++m) {
        if (c[m] >= i) done = true;
        if (!done) s -= a[m] * yv[m];
    }
    if (!done)  // a row with more than kTrsBatch entries below the diagonal
        for (int q = q0 + kTrsBatch; q < q1; ++q) {
            const int k = col[q];
            if (k >= i) break;
            s -= lu[q] * y[k];
        }
    y[i] = s;
}

__device__ __forceinline__ void trs_upper_row(int i, const int *__restrict__ rp, const int *__restrict__ col,
                                              const double *__restrict__ lu, const double *__restrict__ y,
                                              double *z) {
#pragma clang fp contract(off)
    const int q0 = rp[i], q1 = rp[i + 1];
    int c[kTrsBatch];
    double a[kTrsBatch], zv[kTrsBatch];
#pragma unroll
    for (int m = 0; m < kTrsBatch; ++m) {
        const int q = q0 + m;
        const bool in = q < q1;
        c[m] = in ? col[q] : -1;
        a[m] = in ? lu[q] : 0.0;
    }
#pragma unroll
    for (int m = 0; m < kTrsBatch; ++m) zv[m] = c[m] > i ? z[c[m]] : 0.0;
    double s = y[i], d = 0.0;
#pragma unroll
    for (int m = 0; m < kTrsBatch; ++m) {
        if (c[m] > i) s -= a[m] * zv[m];
        else if (c[m] == i) d = a[m];
    }
    for (int q = q0 + kTrsBatch; q < q1; ++q) {
        const int k = col[q];
        if (k > i) s -= lu[q] * z[k];
        else if (k == i) d = lu[q];
    }
    z[i] = s / d;
}

// A row of either substitution from the level-ordered slot layout: position
// t of the schedule holds row i = perm[t]; its strict entries sit at
// slot * n_pad + t, so a level's threads load them with consecutive
// addresses and need no row bounds first (two round trips: entries, then
// dependencies).  Slots are in column order, so the sums are the sequential
// ones.  lower: x_i = b_i - sum l_ik x_k; upper: x_i = (b_i - sum u_ik x_k) / u_ii.
template <bool LOWER>
__device__ __forceinline__ void trs_row_lv(int64_t t, int i, int w, int64_t n_pad, const int *__restrict__ oc,
                                           const double *__restrict__ ov, const double *__restrict__ diag,
                                           const double *__restrict__ b, double *x) {
#pragma clang fp contract(off)
    double s = b[i];
    for (int s0 = 0; s0 < w; s0 += kTrsBatch) {
        int c[kTrsBatch];
        double v[kTrsBatch], xv[kTrsBatch];
#pragma unroll
        for (int m = 0; m < kTrsBatch; ++m) {
            const int slot = s0 + m;
            const bool in = slot < w;
            c[m] = in ? oc[(int64_t)slot * n_pad + t] : -1;
            v[m] = in ? ov[(int64_t)slot * n_pad + t] : 0.0;
        }
#pragma unroll
        for (int m = 0; m < kTrsBatch; ++m) xv[m] = c[m] >= 0 ? x[c[m]] : 0.0;
#pragma unroll
        for (int m = 0; m < kTrsBatch; ++m)
            if (c[m] >= 0) s -= v[m] * xv[m];
    }
    x[i] = LOWER ? s : s / diag[t];
}

// Packs one triangle's strict entries (and diag(U)) in level order.
__global__ void k_trs_pack(int64_t n, int64_t n_pad, const int *__restrict__ perm, const int *__restrict__ rp,
                           const int *__restrict__ col, const double *__restrict__ lu, int w, int lower,
                           int *__restrict__ oc, double *__restrict__ ov, double *__restrict__ odiag) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    const int i = perm[t];
    int a = 0;
    for (int q = rp[i]; q < rp[i + 1]; ++q) {
        const int c = col[q];
        if (lower ? c < i : c > i) {
            oc[(int64_t)a * n_pad + t] = c;
            ov[(int64_t)a * n_pad + t] = lu[q];
            ++a;
        } else if (!lower && c == i) {
            odiag[t] = lu[q];
        }
    }
    for (; a < w; ++a) {
        oc[(int64_t)a * n_pad + t] = -1;
        ov[(int64_t)a * n_pad + t] = 0.0;
    }
}

__global__ void k_trs_lower_lv(int64_t cnt, int64_t t0, int w, int64_t n_pad, const int *__restrict__ perm,
                               const int *__restrict__ oc, const double *__restrict__ ov,
                               const double *__restrict__ r, double *y) {
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= cnt) return;
    trs_row_lv<true>(t0 + g, perm[t0 + g], w, n_pad, oc, ov, nullptr, r, y);
}

__global__ void k_trs_upper_lv(int64_t cnt, int64_t t0, int w, int64_t n_pad, const int *__restrict__ perm,
                               const int *__restrict__ oc, const double *__restrict__ ov,
                               const double *__restrict__ diag, const double *__restrict__ y, double *z) {
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= cnt) return;
    trs_row_lv<false>(t0 + g, perm[t0 + g], w, n_pad, oc, ov, diag, y, z);
}

// Exact substitution, one level of rows at a time (the rows of a level
// depend only on rows of earlier levels).
__global__ void k_trs_lower_level(int64_t cnt, const int *__restrict__ perm, const int *__restrict__ rp,
                                  const int *__restrict__ col, const double *__restrict__ lu,
                                  const double *__restrict__ r, double *y) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= cnt) return;
    trs_lower_row(perm[t], rp, col, lu, r, y);
}

__global__ void k_trs_upper_level(int64_t cnt, const int *__restrict__ perm, const int *__restrict__ rp,
                                  const int *__restrict__ col, const double *__restrict__ lu,
                                  const double *__restrict__ y, double *z) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= cnt) return;
    trs_upper_row(perm[t], rp, col, lu, y, z);
}

// A run of consecutive small levels solved by one workgroup in one launch:
// level after level, every thread takes rows of the level, and a workgroup
// barrier separates the levels (a row's dependencies lie in earlier levels,
// whose values the barrier makes visible).  Each row does exactly the
// operations of the one-level kernels, so results are the same bit for bit.
constexpr int kTrsRunWG = 1024;       // threads of the run kernels
constexpr int64_t kTrsSmall = 1024;   // levels of at most this many rows join a run

__global__ __launch_bounds__(kTrsRunWG) void k_trs_lower_run(int l0, int l1, const int64_t *__restrict__ ptr,
                                                             const int *__restrict__ perm,
                                                             const int *__restrict__ rp, const int *__restrict__ col,
                                                             const double *__restrict__ lu,
                                                             const double *__restrict__ r, double *y) {
    for (int l = l0; l < l1; ++l) {
        const int64_t b = ptr[l], e = ptr[l + 1];
        for (int64_t t = b + threadIdx.x; t < e; t += kTrsRunWG) trs_lower_row(perm[t], rp, col, lu, r, y);
        __syncthreads();
    }
}

__global__ __launch_bounds__(kTrsRunWG) void k_trs_upper_run(int l0, int l1, const int64_t *__restrict__ ptr,
                                                             const int *__restrict__ perm,
                                                             const int *__restrict__ rp, const int *__restrict__ col,
                                                             const double *__restrict__ lu,
                                                             const double *__restrict__ y, double *z) {
    for (int l = l0; l < l1; ++l) {
        const int64_t b = ptr[l], e = ptr[l + 1];
        for (int64_t t = b + threadIdx.x; t < e; t += kTrsRunWG) trs_upper_row(perm[t], rp, col, lu, y, z);
        __syncthreads();
    }
}

__global__ __launch_bounds__(kTrsRunWG) void k_trs_lower_run_lv(int l0, int l1, const int64_t *__restrict__ ptr,
                                                                const int *__restrict__ perm, int w, int64_t n_pad,
                                                                const int *__restrict__ oc,
                                                                const double *__restrict__ ov,
                                                                const double *__restrict__ r, double *y) {
    for (int l = l0; l < l1; ++l) {
        const int64_t b = ptr[l], e = ptr[l + 1];
        for (int64_t t = b + threadIdx.x; t < e; t += kTrsRunWG) trs_row_lv<true>(t, perm[t], w, n_pad, oc, ov, nullptr, r, y);
        __syncthreads();
    }
}

__global__ __launch_bounds__(kTrsRunWG) void k_trs_upper_run_lv(int l0, int l1, const int64_t *__restrict__ ptr,
                                                                const int *__restrict__ perm, int w, int64_t n_pad,
                                                                const int *__restrict__ oc,
                                                                const double *__restrict__ ov,
                                                                const double *__restrict__ diag,
                                                                const double *__restrict__ y, double *z) {
    for (int l = l0; l < l1; ++l) {
        const int64_t b = ptr[l], e = ptr[l + 1];
        for (int64_t t = b + threadIdx.x; t < e; t += kTrsRunWG) trs_row_lv<false>(t, perm[t], w, n_pad, oc, ov, diag, y, z);
        __syncthreads();
    }
}

// Launch schedule of one triangle: maximal runs of consecutive levels with
// at most kTrsSmall rows become one entry (one launch of a run kernel);
// every other level is an entry of its own (a one-level launch).
static std::vector<int2> trs_runs(const std::vector<int64_t> &ptr) {
    std::vector<int2> out;
    const int nl = (int)ptr.size() - 1;
    int l = 0;
    while (l < nl) {
        int e = l;
        while (e < nl && ptr[e + 1] - ptr[e] <= kTrsSmall) ++e;
        if (e - l >= 2) {
            out.push_back(make_int2(l, e));
            l = e;
        } else {
            out.push_back(make_int2(l, l + 1));
            ++l;
        }
    }
    return out;
}

// One Jacobi sweep on L y = r (unit diagonal): yout_i = r_i - sum_{k<i} l_ik yin_k.
__global__ void k_trs_jlower(int64_t n, const int *__restrict__ rp, const int *__restrict__ col,
                             const double *__restrict__ lu, const double *__restrict__ r,
                             const double *__restrict__ yin, double *__restrict__ yout) {
#pragma clang fp contract(off)
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double s = r[i];
    for (int64_t q = rp[i]; q < rp[i + 1]; ++q) {
        const int k = col[q];
        if (k >= i) break;
        s -= lu[q] * yin[k];
    }
    yout[i] = s;
}

// One Jacobi sweep on U z = y: zout_i = (y_i - sum_{k>i} u_ik zin_k) / u_ii;
// zin = nullptr is the zeroth sweep z = y / u_ii.
__global__ void k_trs_jupper(int64_t n, const int *__restrict__ rp, const int *__restrict__ col,
                             const double *__restrict__ lu, const int *__restrict__ dpos,
                             const double *__restrict__ y, const double *__restrict__ zin,
                             double *__restrict__ zout) {
#pragma clang fp contract(off)
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    if (!zin) {
        zout[i] = y[i] / lu[dpos[i]];
        return;
    }
    double s = y[i], d = 0.0;
    for (int64_t q = rp[i]; q < rp[i + 1]; ++q) {
        const int k = col[q];
        if (k > i) s -= lu[q] * zin[k];
        else if (k == i) d = lu[q];
    }
    zout[i] = s / d;
}

// The factors repacked for the Jacobi sweeps: strictly lower and strictly
// upper entries in slot-major arrays [w][n_pad] (slot s of row i at
// s n_pad + i, in the row's ascending column order; column -1 pads), and
// the diagonal of U.  A wave's loads of one slot are contiguous.
__global__ void k_ilu_split(int64_t n, int64_t n_pad, const int *__restrict__ rp, const int *__restrict__ col,
                            const double *__restrict__ lu, int wl, int wu, int *__restrict__ lcol,
                            double *__restrict__ lval, int *__restrict__ ucol, double *__restrict__ uval,
                            double *__restrict__ udiag) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int a = 0, b = 0;
    for (int64_t q = rp[i]; q < rp[i + 1]; ++q) {
        const int c = col[q];
        if (c < i) {
            lcol[(int64_t)a * n_pad + i] = c;
            lval[(int64_t)a * n_pad + i] = lu[q];
            ++a;
        } else if (c > i) {
            ucol[(int64_t)b * n_pad + i] = c;
            uval[(int64_t)b * n_pad + i] = lu[q];
            ++b;
        } else {
            udiag[i] = lu[q];
        }
    }
    for (; a < wl; ++a) {
        lcol[(int64_t)a * n_pad + i] = -1;
        lval[(int64_t)a * n_pad + i] = 0.0;
    }
    for (; b < wu; ++b) {
        ucol[(int64_t)b * n_pad + i] = -1;
        uval[(int64_t)b * n_pad + i] = 0.0;
    }
}

// One Jacobi sweep on a triangle in the slot-major layout:
// out_i = (rhs_i - sum_s val_s in[col_s]) [/ diag_i]; in = nullptr: out = rhs [/ diag].
__global__ __launch_bounds__(256) void k_trs_jsweep(int64_t n, int64_t n_pad, int w, const int *__restrict__ tcol,
                                                    const double *__restrict__ tval,
                                                    const double *__restrict__ diag,
                                                    const double *__restrict__ rhs,
                                                    const double *__restrict__ in, double *__restrict__ out) {
#pragma clang fp contract(off)
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double s = rhs[i];
    if (in) {
        for (int k = 0; k < w; ++k) {
            const int c = __builtin_nontemporal_load(tcol + (int64_t)k * n_pad + i);
            if (c < 0) break;
            s -= __builtin_nontemporal_load(tval + (int64_t)k * n_pad + i) * in[c];
        }
    }
    out[i] = diag ? s / diag[i] : s;
}

// out = alpha t + beta out (beta == 0 overwrites).
__global__ void k_ilu_axpby(int64_t n, double alpha, const double *__restrict__ t, double beta,
                            double *__restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    out[i] = beta == 0.0 ? alpha * t[i] : alpha * t[i] + beta * out[i];
}

static unsigned blocks(int64_t n) { return (unsigned)((n + 255) / 256 > 0 ? (n + 255) / 256 : 1); }

hipError_t ilu_apply(const IluImpl &P, double alpha, const void *r, double beta, void *out, hipStream_t s) {
    const MatrixImpl &A = *P.A;
    const int64_t n = A.nrows;
    if (P.chain) return ilu_chain_apply(P, alpha, (const double *)r, beta, (double *)out, s);
    const int *rp = (const int *)A.row_ptr->p, *col = (const int *)A.col->p;
    const double *lu = (const double *)P.lu->p;
    const int *dpos = (const int *)P.dpos->p;
    double *y = (double *)P.y->p, *t = (double *)P.t->p, *z = (double *)P.z->p;
    const double *rr = (const double *)r;
    if (P.trisolve == 0 && P.lcol_lv) {
        const int *lp = (const int *)P.lperm->p, *up = (const int *)P.uperm->p;
        const int64_t *lpd = (const int64_t *)P.lptr_d->p, *upd = (const int64_t *)P.uptr_d->p;
        const int64_t np = P.n_pad;
        const int *lc = (const int *)P.lcol_lv->p, *uc = (const int *)P.ucol_lv->p;
        const double *lv = (const double *)P.lval_lv->p, *uv = (const double *)P.uval_lv->p;
        const double *ud = (const double *)P.udiag_lv->p;
        for (const int2 &g : P.lruns) {
            if (g.y - g.x > 1) {
                hipLaunchKernelGGL(k_trs_lower_run_lv, dim3(1), dim3(kTrsRunWG), 0, s, g.x, g.y, lpd, lp, P.lw_lv, np,
                                   lc, lv, rr, y);
            } else {
                const int64_t c = P.lptr[g.x + 1] - P.lptr[g.x];
                hipLaunchKernelGGL(k_trs_lower_lv, dim3(blocks(c)), dim3(256), 0, s, c, P.lptr[g.x], P.lw_lv, np, lp,
                                   lc, lv, rr, y);
            }
        }
        for (const int2 &g : P.uruns) {
            if (g.y - g.x > 1) {
                hipLaunchKernelGGL(k_trs_upper_run_lv, dim3(1), dim3(kTrsRunWG), 0, s, g.x, g.y, upd, up, P.uw_lv, np,
                                   uc, uv, ud, (const double *)y, z);
            } else {
                const int64_t c = P.uptr[g.x + 1] - P.uptr[g.x];
                hipLaunchKernelGGL(k_trs_upper_lv, dim3(blocks(c)), dim3(256), 0, s, c, P.uptr[g.x], P.uw_lv, np, up,
                                   uc, uv, ud, (const double *)y, z);
            }
        }
    } else if (P.trisolve == 0) {
        const int *lp = (const int *)P.lperm->p, *up = (const int *)P.uperm->p;
        const int64_t *lpd = (const int64_t *)P.lptr_d->p, *upd = (const int64_t *)P.uptr_d->p;
        for (const int2 &g : P.lruns) {
            if (g.y - g.x > 1) {
                hipLaunchKernelGGL(k_trs_lower_run, dim3(1), dim3(kTrsRunWG), 0, s, g.x, g.y, lpd, lp, rp, col, lu, rr,
                                   y);
            } else {
                const int64_t c = P.lptr[g.x + 1] - P.lptr[g.x];
                hipLaunchKernelGGL(k_trs_lower_level, dim3(blocks(c)), dim3(256), 0, s, c, lp + P.lptr[g.x], rp,
                                   col, lu, rr, y);
            }
        }
        for (const int2 &g : P.uruns) {
            if (g.y - g.x > 1) {
                hipLaunchKernelGGL(k_trs_upper_run, dim3(1), dim3(kTrsRunWG), 0, s, g.x, g.y, upd, up, rp, col, lu,
                                   (const double *)y, z);
            } else {
                const int64_t c = P.uptr[g.x + 1] - P.uptr[g.x];
                hipLaunchKernelGGL(k_trs_upper_level, dim3(blocks(c)), dim3(256), 0, s, c, up + P.uptr[g.x], rp,
                                   col, lu, (const double *)y, z);
            }
        }
    } else {
        // L y = r: y0 = r, then sweeps; U z = y: z0 = y / u_ii, then sweeps
        const bool split = P.lcol != nullptr;
        const int *lc = split ? (const int *)P.lcol->p : nullptr, *uc = split ? (const int *)P.ucol->p : nullptr;
        const double *lv = split ? (const double *)P.lval->p : nullptr;
        const double *uv = split ? (const double *)P.uval->p : nullptr;
        const double *ud = split ? (const double *)P.udiag->p : nullptr;
        const double *yin = rr;
        double *ya = y, *yb = t;
        for (int k = 0; k < P.trs_sweeps; ++k) {
            if (split)
                hipLaunchKernelGGL(k_trs_jsweep, dim3(blocks(n)), dim3(256), 0, s, n, P.n_pad, P.wl, lc, lv,
                                   (const double *)nullptr, rr, yin, ya);
            else
                hipLaunchKernelGGL(k_trs_jlower, dim3(blocks(n)), dim3(256), 0, s, n, rp, col, lu, rr, yin, ya);
            yin = ya;
            std::swap(ya, yb);
        }
        // yin holds L^{-1} r (r itself after zero sweeps); the upper sweeps
        // alternate between z and the free buffer
        double *za = z, *zb = (yin == y) ? t : y;
        if (split)
            hipLaunchKernelGGL(k_trs_jsweep, dim3(blocks(n)), dim3(256), 0, s, n, P.n_pad, P.wu, uc, uv, ud, yin,
                               (const double *)nullptr, za);
        else
            hipLaunchKernelGGL(k_trs_jupper, dim3(blocks(n)), dim3(256), 0, s, n, rp, col, lu, dpos, yin,
                               (const double *)nullptr, za);
        for (int k = 0; k < P.trs_sweeps; ++k) {
            if (split)
                hipLaunchKernelGGL(k_trs_jsweep, dim3(blocks(n)), dim3(256), 0, s, n, P.n_pad, P.wu, uc, uv, ud,
                                   yin, (const double *)za, zb);
            else
                hipLaunchKernelGGL(k_trs_jupper, dim3(blocks(n)), dim3(256), 0, s, n, rp, col, lu, dpos, yin,
                                   (const double *)za, zb);
            std::swap(za, zb);
        }
        z = za;
    }
    hipLaunchKernelGGL(k_ilu_axpby, dim3(blocks(n)), dim3(256), 0, s, n, alpha, (const double *)z, beta,
                       (double *)out);
    return hipGetLastError();
}

}  // namespace mxl

using namespace mxl;

// Longest strictly lower and strictly upper part of any row (the slot
// counts of the split layout), reduced with integer atomics.
__global__ void k_ilu_widths(int64_t n, const int *__restrict__ rp, const int *__restrict__ col,
                             int *__restrict__ w2) {
    int wl = 0, wu = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        int a = 0, b = 0;
        for (int q = rp[i]; q < rp[i + 1]; ++q) {
            const int c = col[q];
            if (c < i) ++a;
            else if (c > i) ++b;
        }
        wl = a > wl ? a : wl;
        wu = b > wu ? b : wu;
    }
    wl = wave_max(wl);
    wu = wave_max(wu);
    if (threadIdx.x % kWave == 0) {
        atomicMax(w2, wl);
        atomicMax(w2 + 1, wu);
    }
}

// Dependency levels of both triangles, computed on the host from the row
// structure (exact triangular solves, and mxl_ilu_info on request).
static mxl_status ilu_levels(IluImpl &P) {
    const MatrixImpl &A = *P.A;
    const int64_t n = A.nrows, nnz = A.nnz;
    hipStream_t s = A.ctx->stream;
    std::vector<int> hrp((size_t)n + 1), hcol((size_t)nnz);
    if (hipMemcpyAsync(hrp.data(), A.row_ptr->p, (n + 1) * 4, hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipMemcpyAsync(hcol.data(), A.col->p, nnz * 4, hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return set_error(MXL_ERR_DEVICE, "ILU structure read-back");
    std::vector<int> lperm, uperm;
    ilu_levels_host(hrp, hcol, true, lperm, P.lptr);
    ilu_levels_host(hrp, hcol, false, uperm, P.uptr);
    // every offset the level launches will take comes from these arrays
    if (!ilu_levels_valid(hrp, hcol, true, lperm, P.lptr) || !ilu_levels_valid(hrp, hcol, false, uperm, P.uptr)) {
        P.lptr.clear();
        P.uptr.clear();
        return set_error(MXL_ERR_INTERNAL, "ILU level schedule failed its invariants");
    }
    // one allocation and, where the lists are small, one copy: a small system's
    // generation is host calls
    Arena lists;
    lists.want(P.lptr_d, P.lptr.size() * 8);
    lists.want(P.uptr_d, P.uptr.size() * 8);
    lists.want(P.lperm, (size_t)n * 4);
    lists.want(P.uperm, (size_t)n * 4);
    if (!lists.alloc()) return set_error(MXL_ERR_OUT_OF_MEMORY, "ILU levels");
    char *base = (char *)P.lptr_d->p;
    const size_t total = (size_t)((char *)P.uperm->p - base) + (size_t)n * 4;
    std::vector<char> stage(total <= (64 << 10) ? total : 0);
    hipError_t e = hipSuccess;
    auto put = [&](const BufPtr &d, const void *src, size_t bytes) {
        if (!stage.empty()) memcpy(stage.data() + ((char *)d->p - base), src, bytes);
        else if (e == hipSuccess) e = hipMemcpyAsync(d->p, src, bytes, hipMemcpyHostToDevice, s);
    };
    put(P.lptr_d, P.lptr.data(), P.lptr.size() * 8);
    put(P.uptr_d, P.uptr.data(), P.uptr.size() * 8);
    put(P.lperm, lperm.data(), (size_t)n * 4);
    put(P.uperm, uperm.data(), (size_t)n * 4);
    if (!stage.empty()) e = hipMemcpyAsync(base, stage.data(), total, hipMemcpyHostToDevice, s);
    if (e != hipSuccess || hipStreamSynchronize(s) != hipSuccess)
        return set_error(MXL_ERR_DEVICE, "ILU levels upload");
    P.lruns = trs_runs(P.lptr);
    P.uruns = trs_runs(P.uptr);
    int wl = 0, wu = 0;
    for (int64_t i = 0; i < n; ++i) {
        int a = 0, b = 0;
        for (int q = hrp[(size_t)i]; q < hrp[(size_t)i + 1]; ++q) {
            const int c = hcol[(size_t)q];
            if (c < i) ++a;
            else if (c > i) ++b;
        }
        wl = std::max(wl, a);
        wu = std::max(wu, b);
    }
    P.lw_lv = wl;
    P.uw_lv = wu;
    return MXL_OK;
}

// The level-ordered slot layout of both triangles (exact solves), built
// from the final factors; skipped (the solves walk CSR rows) when its
// padding would exceed 4x the factor storage.
static mxl_status ilu_pack_levels(IluImpl &P) {
    const MatrixImpl &A = *P.A;
    const int64_t n = A.nrows, nnz = A.nnz;
    const int64_t n_pad = (n + 63) / 64 * 64;
    if ((int64_t)(P.lw_lv + P.uw_lv) * n_pad > 4 * nnz + 2 * n) return MXL_OK;
    const int wl = P.lw_lv, wu = P.uw_lv;
    BufPtr lc, lv, uc, uv, ud;
    Arena a;
    a.want(lv, (size_t)wl * n_pad * 8);
    a.want(uv, (size_t)wu * n_pad * 8);
    a.want(ud, (size_t)n * 8);
    a.want(lc, (size_t)wl * n_pad * 4);
    a.want(uc, (size_t)wu * n_pad * 4);
    if (!a.alloc()) return set_error(MXL_ERR_OUT_OF_MEMORY, "ILU level-ordered factors");
    hipStream_t s = A.ctx->stream;
    const int *rp = (const int *)A.row_ptr->p, *col = (const int *)A.col->p;
    const double *lu = (const double *)P.lu->p;
    hipLaunchKernelGGL(k_trs_pack, dim3(blocks(n)), dim3(256), 0, s, n, n_pad, (const int *)P.lperm->p, rp, col, lu,
                       wl, 1, (int *)lc->p, (double *)lv->p, (double *)nullptr);
    hipLaunchKernelGGL(k_trs_pack, dim3(blocks(n)), dim3(256), 0, s, n, n_pad, (const int *)P.uperm->p, rp, col, lu,
                       wu, 0, (int *)uc->p, (double *)uv->p, (double *)ud->p);
    hipError_t e;
    if ((e = hipGetLastError()) != hipSuccess || (e = hipStreamSynchronize(s)) != hipSuccess)
        return set_error(MXL_ERR_DEVICE, std::string("ILU level pack: ") + hipGetErrorString(e));
    P.n_pad = n_pad;
    P.lcol_lv = lc;
    P.lval_lv = lv;
    P.ucol_lv = uc;
    P.uval_lv = uv;
    P.udiag_lv = ud;
    return MXL_OK;
}

extern "C" mxl_status mxl_ilu_generate(const mxl_op *Aop, int32_t sweeps, int32_t trisolve, int32_t trs_sweeps,
                                       mxl_op **Pout) try {
    if (!Aop || !Pout || Aop->kind != MXL_OP_MATRIX)
        return set_error(MXL_ERR_INVALID_ARG, "matrix operator and output required");
    *Pout = nullptr;
    if (sweeps < 0 || trs_sweeps < 0 || (trisolve != 0 && trisolve != 1))
        return set_error(MXL_ERR_INVALID_ARG, "sweeps >= 0, trisolve 0 or 1, trs_sweeps >= 0");
    const auto &A = Aop->mat;
    if (A->nrows != A->ncols) return set_error(MXL_ERR_NOT_IMPLEMENTED, "ILU needs a square matrix");
    if (A->dtype != MXL_F64) return set_error(MXL_ERR_NOT_IMPLEMENTED, "ILU needs an FP64 matrix");
    if (A->format == MXL_FMT_STENCIL) return set_error(MXL_ERR_NOT_IMPLEMENTED, "ILU needs stored matrix rows");
    if (A->nrows == 0) return set_error(MXL_ERR_INVALID_ARG, "empty matrix");
    DeviceScope ds(A->ctx->device);
    hipStream_t s = A->ctx->stream;
    const int64_t n = A->nrows, nnz = A->nnz;
    auto P = std::make_shared<IluImpl>();
    P->A = A;
    P->sweeps = sweeps;
    P->trisolve = trisolve;
    P->trs_sweeps = trs_sweeps;
    // Allocations are few and as small as they can be: one of 90 MB costs 50 us,
    // its release 300.  Exact solves run along the rows' chains where they form
    // some (planned on the device from the pattern, no host copy of the matrix: a new
    // 101^3 system 33 -> 1.6 ms); the sweeps' second copy of the factors and their row
    // indices then stand where the packed factors will.  Without memory for the plan or
    // the packed factors the solves run by levels, for which the plan's is given back.
    BufPtr head, old;
    Arena tmp, keep, plan, packed;
    ChainPlan chains;
    keep.want(head, chain_head_bytes());
    keep.want(P->dpos, (size_t)n * 4);
    keep.want(P->y, (size_t)n * 8);
    keep.want(P->z, (size_t)n * 8);
    if (!keep.alloc()) return set_error(MXL_ERR_OUT_OF_MEMORY, "ILU workspace");
    bool chain = false;
    if (trisolve == 0) {
        chain_plan_want(chains, n, plan);
        chain = plan.alloc();
    }
    const int *rp = (const int *)A->row_ptr->p, *col = (const int *)A->col->p;
    const double *val = (const double *)A->val->p;
    int hb = INT_MAX, *bad, *w2;
    hipError_t e;
    mxl_status lst;
    if ((e = chain_head_init(head, bad, w2, s)) != hipSuccess) return set_error(MXL_ERR_DEVICE, hipGetErrorString(e));
    hipLaunchKernelGGL(k_ilu_diag, dim3(blocks(n)), dim3(256), 0, s, n, rp, col, val, (int *)P->dpos->p, bad);
    if ((e = hipGetLastError()) != hipSuccess || (chain && (e = chain_gather(*P, chains, head)) != hipSuccess))
        return set_error(MXL_ERR_DEVICE, std::string("ILU set-up: ") + hipGetErrorString(e));
    if ((lst = chain_read(*P, chains, head, hb, chain)) != MXL_OK) return lst;
    if (hb != INT_MAX) {
        char msg[96];
        snprintf(msg, sizeof msg, "row %d has a missing or zero diagonal", hb);
        return set_error(MXL_ERR_ZERO_DIAG, msg);
    }
    const size_t old_bytes = ((size_t)nnz * 8 + 255) / 256 * 256, sweep_bytes = old_bytes + (size_t)nnz * 4;
    void *old_p, *row_p;
    if (chain) {
        BufPtr rest;  // keeps the sweeps' arrays inside the allocation
        packed.want(P->lu, (size_t)nnz * 8);
        packed.want(P->tickets, 12);
        const size_t have = chain_want(*P, chains, packed);
        packed.want(rest, have < sweep_bytes ? sweep_bytes - have : 0);
        chain = packed.alloc();
        if (chain) old_p = P->lo.code->p;
    }
    if (!chain) {
        chains = ChainPlan();
        tmp.want(old, sweep_bytes);
        keep.want(P->lu, (size_t)nnz * 8);
        keep.want(P->t, (size_t)n * 8);
        if (!tmp.alloc() || !keep.alloc()) return set_error(MXL_ERR_OUT_OF_MEMORY, "ILU workspace");
        old_p = old->p;
    }
    row_p = (char *)old_p + old_bytes;
    if ((e = launch_csr_to_coo(*A, (int *)row_p, s)) != hipSuccess)
        return set_error(MXL_ERR_DEVICE, std::string("ILU set-up: ") + hipGetErrorString(e));
    // factors: initial guess, then the sweeps (ping-pong, the result in P->lu)
    double *cur = (double *)(sweeps % 2 == 0 ? P->lu->p : old_p);
    double *nxt = (double *)(sweeps % 2 == 0 ? old_p : P->lu->p);
    hipLaunchKernelGGL(k_ilu_init, dim3(blocks(nnz)), dim3(256), 0, s, nnz, (const int *)row_p, col, val,
                       (const int *)P->dpos->p, cur);
    for (int k = 0; k < sweeps; ++k) {
        hipLaunchKernelGGL(k_parilu_sweep, dim3(blocks(nnz)), dim3(256), 0, s, nnz, rp, (const int *)row_p, col,
                           val, (const int *)P->dpos->p, (const double *)cur, nxt);
        std::swap(cur, nxt);
    }
    if ((e = hipGetLastError()) != hipSuccess) return set_error(MXL_ERR_DEVICE, hipGetErrorString(e));
    // other exact solves run over the dependency levels (built on the host)
    if (chain && (lst = chain_pack(*P, chains)) != MXL_OK) return lst;
    if (trisolve == 0 && !chain && (lst = ilu_levels(*P)) != MXL_OK) return lst;
    if (trisolve == 0 && !chain && (lst = ilu_pack_levels(*P)) != MXL_OK) return lst;
    // Jacobi sweeps read the factors repacked slot-major when the padding
    // stays within 4x the factor storage
    if (trisolve == 1) {
        int hw[2] = {0, 0};
        hipLaunchKernelGGL(k_ilu_widths, dim3((unsigned)std::min<int64_t>(blocks(n), 2048)), dim3(256), 0, s, n, rp,
                           col, w2);
        if (hipMemcpyAsync(hw, w2, 8, hipMemcpyDeviceToHost, s) != hipSuccess || hipStreamSynchronize(s) != hipSuccess)
            return set_error(MXL_ERR_DEVICE, "ILU widths read-back");
        const int wl = hw[0], wu = hw[1];
        const int64_t n_pad = (n + 63) / 64 * 64;
        if ((int64_t)(wl + wu) * n_pad <= 4 * nnz + 2 * n) {
            P->wl = wl;
            P->wu = wu;
            P->n_pad = n_pad;
            keep.want(P->lcol, (size_t)wl * n_pad * 4);
            keep.want(P->lval, (size_t)wl * n_pad * 8);
            keep.want(P->ucol, (size_t)wu * n_pad * 4);
            keep.want(P->uval, (size_t)wu * n_pad * 8);
            keep.want(P->udiag, (size_t)n * 8);
            if (!keep.alloc())
                return set_error(MXL_ERR_OUT_OF_MEMORY, "ILU split factors");
            hipLaunchKernelGGL(k_ilu_split, dim3(blocks(n)), dim3(256), 0, s, n, n_pad, rp, col,
                               (const double *)P->lu->p, wl, wu, (int *)P->lcol->p, (double *)P->lval->p,
                               (int *)P->ucol->p, (double *)P->uval->p, (double *)P->udiag->p);
            if ((e = hipGetLastError()) != hipSuccess || (e = hipStreamSynchronize(s)) != hipSuccess)
                return set_error(MXL_ERR_DEVICE, std::string("ILU split: ") + hipGetErrorString(e));
        }
    }
    auto *op = new mxl_op;
    op->kind = MXL_OP_ILU;
    op->ilu = P;
    *Pout = op;
    return MXL_OK;
} catch (...) {
    return mxl::abi_exception(__func__);
}

extern "C" mxl_status mxl_ilu_info(const mxl_op *Pop, double *lu_host, int32_t *levels_host) try {
    if (!Pop || Pop->kind != MXL_OP_ILU) return set_error(MXL_ERR_INVALID_ARG, "not an ILU operator");
    const IluImpl &P = *Pop->ilu;
    DeviceScope ds(P.A->ctx->device);
    hipStream_t s = P.A->ctx->stream;
    if (levels_host && P.lptr.empty()) {  // Jacobi-sweep factors: levels only on request
        mxl_status lst = ilu_levels(const_cast<IluImpl &>(P));
        if (lst != MXL_OK) return lst;
    }
    if (levels_host) {
        levels_host[0] = (int32_t)(P.lptr.size() - 1);
        levels_host[1] = (int32_t)(P.uptr.size() - 1);
    }
    if (lu_host) {
        if (hipMemcpyAsync(lu_host, P.lu->p, (size_t)P.A->nnz * 8, hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess)
            return set_error(MXL_ERR_DEVICE, "copy ILU factors");
    }
    return P.chain ? ilu_chain_check(P) : MXL_OK;
} catch (...) {
    return mxl::abi_exception(__func__);
}
