// Explicit inverse of the coarsest operator (Section 2, coarse level solver)
// by in-place Gauss-Jordan elimination with partial pivoting: in step k the
// row with the largest |value| in column k among the rows not yet used
// (lowest row on ties) becomes the pivot row p_k, every other row loses its
// multiple of it, and column k takes the column of the accumulated
// transformation.  Rows stay in place; at the end S = T in place with
// inverse(k, p_k') = S(p_k, k').  Rows not yet used see the operations of LU
// with partial pivoting.
//
// Up to 128 rows one workgroup inverts a system straight from its CSR rows,
// the matrix in registers (4 x 4 entries a thread); all systems of a batch go
// in one launch.  What bounds it is the chain of steps: two barriers, a
// maximum over the column and a division each, 1.2 us (80 us for up to 64 rows).
// Larger systems take panels of 16 (8) columns: one workgroup with a thread per
// row eliminates the panel in registers (30 us), then the whole grid adds the
// panel's transformation to the other columns (10 us).
//
// Blocked LU with the panel in LDS and a separate inverse by substitution took
// 270 us for 64 rows and 1.6 ms for 205 (0.56 ms now); a batch of 32 systems
// went through it one system after the other, 7 ms of a 16.4 ms pass.
#include <cstdint>

#include "amg_device.hpp"
#include "amg_internal.hpp"

namespace amg {

namespace {
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_max(double x) {
    const int lo = __double2loint(x), hi = __double2hiint(x);
    const int l2 = __builtin_amdgcn_update_dpp(lo, lo, CTRL, ROWS, 0xf, false);
    const int h2 = __builtin_amdgcn_update_dpp(hi, hi, CTRL, ROWS, 0xf, false);
    return fmax(x, __hiloint2double(h2, l2));
}

// Maximum over the wave, in every lane (NaN ignored).
__device__ __forceinline__ double wave_max(double x) {
    x = dpp_max<0x111, 0xf>(x);  // row_shr 1, 2, 4, 8: lane 15 of each row of 16
    x = dpp_max<0x112, 0xf>(x);
    x = dpp_max<0x114, 0xf>(x);
    x = dpp_max<0x118, 0xf>(x);
    x = dpp_max<0x142, 0xa>(x);  // row_bcast 15, 31: lane 63
    x = dpp_max<0x143, 0xc>(x);
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), kWave - 1),
                            __builtin_amdgcn_readlane(__double2loint(x), kWave - 1));
}

constexpr int kRT = 4;  // entries a thread holds: kRT x kRT
}  // namespace

// One system a workgroup of TX x TX threads, n <= 4 TX.
template <int TX>
__global__ __launch_bounds__(TX* TX) void k_dense_small(DenseJob one, const DenseJob* __restrict__ many) {
    constexpr int M = kRT * TX, NT = TX * TX;
    __shared__ double S[M * M];
    __shared__ double cb[2][M], rb[M];
    __shared__ int prow[M], step[M];
    const DenseJob J = many ? many[blockIdx.x] : one;
    const int n = J.n, tid = threadIdx.x, tx = tid % TX, ty = tid / TX, lane = tid % kWave;
    for (int t = tid; t < n * M; t += NT) S[t] = 0.0;
    __syncthreads();
    for (int i = tid; i < n; i += NT)
        for (int k = J.rp[i]; k < J.rp[i + 1]; ++k) {
            const int c = J.ci[k] + J.col_add;
            if (c >= 0 && c < n) S[i * M + c] = J.v[k];
        }
    __syncthreads();
    double x[kRT][kRT];
#pragma unroll
    for (int a = 0; a < kRT; ++a)
#pragma unroll
        for (int b = 0; b < kRT; ++b) {
            const int i = ty + TX * a, j = tx + TX * b;
            x[a][b] = i < n && j < n ? S[i * M + j] : 0.0;
        }
    bool free0 = lane < n, free1 = M > kWave && lane + kWave < n;
#pragma unroll
    for (int kb = 0; kb < kRT; ++kb) {
#pragma unroll 1
        for (int kx = 0; kx < TX; ++kx) {
            const int k = kx + TX * kb;
            if (k >= n) break;
            double* const c = cb[k & 1];
            if (tx == kx)
#pragma unroll
                for (int a = 0; a < kRT; ++a) c[ty + TX * a] = x[a][kb];
            __syncthreads();
            // every wave finds the pivot by itself
            const double v0 = free0 ? fabs(c[lane]) : -1.0;
            const double v1 = free1 ? fabs(c[(lane + kWave) % M]) : -1.0;
            const double best = wave_max(fmax(v0, v1));
            if (!(best > 0.0) || !isfinite(best)) {  // uniform over the workgroup
                if (tid == 0) atomicOr(J.err, ERR_SINGULAR);
                return;
            }
            const unsigned long long m0 = __ballot(v0 == best), m1 = __ballot(v1 == best);
            const int p = m0 ? __ffsll((long long)m0) - 1 : kWave + __ffsll((long long)m1) - 1;
            if (p == lane) free0 = false;
            if (p == lane + kWave) free1 = false;
            if (ty == p % TX)
#pragma unroll
                for (int a = 0; a < kRT; ++a)
                    if (a == p / TX)
#pragma unroll
                        for (int b = 0; b < kRT; ++b) rb[tx + TX * b] = x[a][b];
            if (tid == 0) {
                prow[k] = p;
                step[p] = k;
            }
            __syncthreads();
            const double piv = c[p];
            double r[kRT];
#pragma unroll
            for (int b = 0; b < kRT; ++b) r[b] = rb[tx + TX * b];
#pragma unroll
            for (int a = 0; a < kRT; ++a) {
                const int i = ty + TX * a;
                if (i == p) {
#pragma unroll
                    for (int b = 0; b < kRT; ++b) x[a][b] = (b == kb && tx == kx ? 1.0 : r[b]) / piv;
                } else {
                    const double f = c[i] / piv;
#pragma unroll
                    for (int b = 0; b < kRT; ++b) x[a][b] = b == kb && tx == kx ? -f : x[a][b] - f * r[b];
                }
            }
        }
    }
    // inverse, column-major, put in order in LDS for coalesced stores
#pragma unroll
    for (int a = 0; a < kRT; ++a)
#pragma unroll
        for (int b = 0; b < kRT; ++b) {
            const int i = ty + TX * a, j = tx + TX * b;
            if (i < n && j < n) S[prow[j] * n + step[i]] = x[a][b];
        }
    __syncthreads();
    for (int t = tid; t < n * n; t += NT) J.ainv_t[t] = S[t];
}

// Panel of W columns from k0: thread tid holds rows tid + NT q.  stp[i]:
// the step that used row i, or -1; prow[k]: the row step k used; pb: the pivot
// rows of the panel (all columns, as they were), for k_dense_update.
template <int W, int RPT, int NT>
__global__ __launch_bounds__(NT) void k_dense_panel(int n, int k0, double* __restrict__ a,
                                                          double* __restrict__ pb, int* __restrict__ prow,
                                                          int* __restrict__ stp, int* err) {
    constexpr int NW = NT / kWave;
    __shared__ double sv[2][NW];
    __shared__ int si[2][NW];
    __shared__ double rowb[W];
    __shared__ int pr[W];
    if (*err & ERR_SINGULAR) return;  // an earlier panel failed (uniform)
    const int tid = threadIdx.x, lane = tid % kWave, wid = tid / kWave;
    const int kb = min(W, n - k0);
    double w[RPT][W];
    bool live[RPT];
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int i = tid + NT * q;
        live[q] = i < n && (k0 == 0 || stp[i] < 0);
        if (i < n && k0 == 0) stp[i] = -1;
#pragma unroll
        for (int c = 0; c < W; ++c) w[q][c] = i < n && c < kb ? a[(size_t)i * n + k0 + c] : 0.0;
    }
    // The columns rotate through the registers, the current one in w[][0], so
    // that the loop stays rolled (unrolled 16 times a panel took 33 us, not 30).
#pragma unroll 1
    for (int c = 0; c < W; ++c) {
        if (c >= kb) {  // columns past the end: only turned into place
#pragma unroll
            for (int q = 0; q < RPT; ++q) {
                const double t = w[q][0];
#pragma unroll
                for (int e = 1; e < W; ++e) w[q][e - 1] = w[q][e];
                w[q][W - 1] = t;
            }
            continue;
        }
        double v = -1.0;
        int at = 0;
#pragma unroll
        for (int q = 0; q < RPT; ++q) {  // rows ascend: strict '>' keeps the lowest
            const double t = live[q] ? fabs(w[q][0]) : -1.0;
            if (t > v) {
                v = t;
                at = q;
            }
        }
        // lowest row with the maximum: by wave, then over the waves
        const double wm = wave_max(v);
        int row = v == wm ? tid + NT * at : INT_MAX;
        if (RPT > 1) {
            for (int o = kWave / 2; o > 0; o >>= 1) row = min(row, __shfl_xor(row, o));
        } else {
            const unsigned long long m = __ballot(v == wm);
            row = m ? wid * kWave + __ffsll((long long)m) - 1 : INT_MAX;
        }
        if (lane == 0) {
            sv[c & 1][wid] = wm;
            si[c & 1][wid] = row;
        }
        __syncthreads();
        const double sw = lane < NW ? sv[c & 1][lane] : -1.0;
        const double best = wave_max(sw);
        if (!(best > 0.0) || !isfinite(best)) {  // uniform
            if (tid == 0) atomicOr(err, ERR_SINGULAR);
            return;
        }
        int p = INT_MAX;
        unsigned long long m = __ballot(lane < NW && sw == best);
        if (RPT == 1) {  // the waves' rows ascend
            p = si[c & 1][__ffsll((long long)m) - 1];
        } else {
            for (; m != 0; m &= m - 1) p = min(p, si[c & 1][__ffsll((long long)m) - 1]);
        }
#pragma unroll
        for (int q = 0; q < RPT; ++q)
            if (tid + NT * q == p) {
                live[q] = false;
                stp[p] = k0 + c;
#pragma unroll
                for (int e = 0; e < W; ++e) rowb[e] = w[q][e];
            }
        if (tid == 0) pr[c] = p;
        __syncthreads();
        const double piv = rowb[0];
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            if (tid + NT * q == p) {
#pragma unroll
                for (int e = 1; e < W; ++e) w[q][e - 1] = w[q][e] / piv;
                w[q][W - 1] = 1.0 / piv;
            } else {
                const double f = w[q][0] / piv;
#pragma unroll
                for (int e = 1; e < W; ++e) w[q][e - 1] = w[q][e] - f * rowb[e];
                w[q][W - 1] = -f;
            }
        }
    }
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int i = tid + NT * q;
        if (i < n)
#pragma unroll
            for (int c = 0; c < W; ++c)
                if (c < kb) a[(size_t)i * n + k0 + c] = w[q][c];
    }
    __syncthreads();
    if (tid < kb) prow[k0 + tid] = pr[tid];
    for (int c = 0; c < kb; ++c)
        for (int j = tid; j < n; j += NT) pb[(size_t)c * n + j] = a[(size_t)pr[c] * n + j];
}

namespace {
constexpr int UPD_T = 64;  // rows and columns of an update block
}

// Every other column j: a(i, j) = (row i is a pivot of this panel ? 0 : a(i, j)) + sum_c W(i, c) pb(c, j).
template <int W>
__global__ __launch_bounds__(256) void k_dense_update(int n, int k0, double* __restrict__ a,
                                                      const double* __restrict__ pb, const int* __restrict__ stp,
                                                      const int* err) {
    __shared__ double w[UPD_T][W];
    __shared__ int used[UPD_T];
    if (*err & ERR_SINGULAR) return;  // uniform
    const int kb = min(W, n - k0), i0 = blockIdx.y * UPD_T, j = blockIdx.x * UPD_T + threadIdx.x % UPD_T;
    for (int t = threadIdx.x; t < UPD_T * W; t += 256) {
        const int i = i0 + t / W, c = t % W;
        w[t / W][c] = i < n && c < kb ? a[(size_t)i * n + k0 + c] : 0.0;
    }
    if (threadIdx.x < UPD_T) {
        const int i = i0 + threadIdx.x;
        used[threadIdx.x] = i < n && stp[i] >= k0 && stp[i] < k0 + kb;
    }
    __syncthreads();
    if (j >= n || (j >= k0 && j < k0 + kb)) return;
    double p[W];
#pragma unroll
    for (int c = 0; c < W; ++c) p[c] = c < kb ? pb[(size_t)c * n + j] : 0.0;
    for (int t = threadIdx.x / UPD_T; t < UPD_T && i0 + t < n; t += 256 / UPD_T) {
        double* const e = a + (size_t)(i0 + t) * n + j;
        double s = used[t] ? 0.0 : *e;
#pragma unroll
        for (int c = 0; c < W; ++c) s += w[t][c] * p[c];
        *e = s;
    }
}

__global__ __launch_bounds__(256) void k_dense_order(int n, const double* __restrict__ a, const int* __restrict__ prow,
                                                     const int* __restrict__ stp, double* __restrict__ ainv_t,
                                                     const int* err) {
    if (*err & ERR_SINGULAR) return;  // the maps are incomplete
    const int j = blockIdx.x * 64 + threadIdx.x % 64;
    for (int i = blockIdx.y * 64 + threadIdx.x / 64; i < min(n, (int)(blockIdx.y + 1) * 64); i += 4)
        if (j < n) ainv_t[(size_t)prow[j] * n + stp[i]] = a[(size_t)i * n + j];
}

__global__ __launch_bounds__(256) void k_dense_assemble(DenseJob J, double* __restrict__ a) {
    const int n = J.n;
    for (int i = blockIdx.x; i < n; i += gridDim.x) {
        for (int c = threadIdx.x; c < n; c += 256) a[(size_t)i * n + c] = 0.0;
        __syncthreads();
        for (int k = J.rp[i] + threadIdx.x; k < J.rp[i + 1]; k += 256) {
            const int c = J.ci[k] + J.col_add;
            if (c >= 0 && c < n) a[(size_t)i * n + c] = J.v[k];
        }
        __syncthreads();
    }
}

void launch_dense_small(const DenseJob& one, const DenseJob* many, int count, int nmax, hipStream_t s) {
    if (count <= 0) return;
    if (nmax <= 64) hipLaunchKernelGGL(k_dense_small<16>, dim3(count), dim3(256), 0, s, one, many);
    else hipLaunchKernelGGL(k_dense_small<32>, dim3(count), dim3(1024), 0, s, one, many);
}

size_t dense_work_doubles(int n) { return n <= kDenseSmall ? 0 : (size_t)n * n + 16 * (size_t)n + (size_t)n; }

void launch_dense_inverse(const DenseJob& J, double* work, hipStream_t s) {
    const int n = J.n;
    if (n <= kDenseSmall) {
        launch_dense_small(J, nullptr, 1, n, s);
        return;
    }
    double* a = work;
    double* pb = a + (size_t)n * n;
    int* prow = reinterpret_cast<int*>(pb + 16 * (size_t)n);
    int* stp = prow + n;
    hipLaunchKernelGGL(k_dense_assemble, dim3(n < 1024 ? n : 1024), dim3(256), 0, s, J, a);
    const dim3 g((n + UPD_T - 1) / UPD_T, (n + UPD_T - 1) / UPD_T);
// one thread a row, while that takes at most 16 waves: fewer waves make the
// panel's barriers cheaper
#define PANELS(W, RPT, NT)                                                                                     \
    for (int k0 = 0; k0 < n; k0 += W) {                                                                        \
        hipLaunchKernelGGL((k_dense_panel<W, RPT, NT>), dim3(1), dim3(NT), 0, s, n, k0, a, pb, prow, stp, J.err); \
        hipLaunchKernelGGL((k_dense_update<W>), g, dim3(256), 0, s, n, k0, a, pb, stp, (const int*)J.err);     \
    }
    if (n <= 256) {
        PANELS(16, 1, 256)
    } else if (n <= 512) {
        PANELS(16, 1, 512)
    } else if (n <= 1024) {
        PANELS(16, 1, 1024)
    } else if (n <= 2048) {
        PANELS(16, 2, 1024)
    } else {
        PANELS(8, 4, 1024)
    }
#undef PANELS
    hipLaunchKernelGGL(k_dense_order, g, dim3(256), 0, s, n, a, prow, stp, J.ainv_t, (const int*)J.err);
}

}  // namespace amg
