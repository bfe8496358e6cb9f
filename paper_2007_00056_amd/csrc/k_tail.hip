// The small levels of the V-cycle in one workgroup.
//
// A level of a few hundred rows costs a kernel each way, 3-5 us for work of a
// fraction of one: the rest is the launch and a chain of dependent loads.  From
// the first level on whose operators, with those of all coarser levels, fit in
// kTailBytes of LDS, the cycle runs in one launch: the operators come in as
// one block packed at setup, loaded all at once together with the right-hand
// side, the coarsest inverse and what the last step needs, and every level's
// steps work in LDS.
//
// The steps are those of the level kernels, in the same order of additions: f_c = P^T (f - w A g) with the
// members in ascending order, g_c = D_c^{-1} f_c; the coarsest solve in double;
// xp = w g + P e, z = xp + w (g - D^{-1} A xp).  Values and sums have the
// preconditioner's type T.
//
// Bound by the chain of LDS reads and instructions of its steps (about 0.8 us a
// step) and 1.5 us for the loads: 428 and 114 rows over 33 take 9.2 us in
// place of five kernels of 3-4 us and their gaps.  A V-cycle on 77 x 45 x 31
// rows in double takes 48.6 us (56.2 with a kernel per step), on
// 61 x 67 x 53 85.5 (96.2), on 64 x 64 17.6 (24.3), on 128^3 160 (170); in single
// precision on 24^3 29.6 (36.5), on 97 x 101 x 89 119 (129).
#include "amg_device.hpp"
#include "amg_internal.hpp"

namespace amg {

namespace {

constexpr int BS = 1024;
constexpr int kStage = 9;        // 16-byte words of the block a thread may load (as 8 or fewer the compiler spills them)
constexpr int kDenseParts = 8, kDenseRows = BS / kDenseParts;
constexpr int kAinvHeld = kDenseRows / kDenseParts;  // entries of the inverse a thread holds, up to 128 coarsest rows
// Most LDS for the cycle.  A level that needs more does not gain: with 902 rows
// and 13,500 entries inside (135 KB) a V-cycle on 24^3 rows takes 31.6 us,
// without them 29.6.
constexpr int kTailBytes = 112 * 1024;

using Word = unsigned __attribute__((ext_vector_type(4)));
// a member of a coarse row: its row and the entries from b up to e
struct alignas(8) Rec {
    uint16_t i, b, e, pad;
};
using Four = int __attribute__((ext_vector_type(4)));

inline int up16(int64_t b) { return (int)((b + 15) & ~int64_t(15)); }

// x of the lane that a row of 16 lanes' data movement names
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double x) {
    return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(x), CTRL, 0xf, 0xf, true),
                            __builtin_amdgcn_mov_dpp(__double2loint(x), CTRL, 0xf, 0xf, true));
}

// A row's sum in the order of the lane-group kernels with 4 (or 8) lanes a row:
// one sum for each of their lanes, over every 4th (8th) entry, and the sums
// added pairwise as a butterfly adds them.  One lane holds four of the sums;
// with 8 a neighbour holds the other four, and both get the row's.  The four
// entries of a step are loaded together (past the row's end the last one
// again, not added): a chain of LDS reads per step, not per entry.
//
// STREAM: the order of the CSR-stream kernels instead, one lane a row: rounded
// products added in entry order.
template <bool STREAM, class T>
__device__ __forceinline__ T tail_row(const T* v, const uint16_t* ci, const T* x, int b, int e, int lane, int lpr) {
    if constexpr (STREAM) {
#pragma clang fp contract(off)
        T s = T(0);
        for (int k = b; k < e; k += 4) {
            T p[4];
            int c[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = min(k + u, e - 1);
                p[u] = v[i];
                c[u] = ci[i];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) p[u] = p[u] * x[c[u]];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const T t = s + p[u];
                s = k + u < e ? t : s;
            }
        }
        return s;
    }
    T s[4] = {T(0), T(0), T(0), T(0)};
    for (int k = b + lane; k < e; k += 4 * lpr) {
        T p[4];
        int c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = min(k + u * lpr, e - 1);
            p[u] = v[i];
            c[u] = ci[i];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const T t = fma(p[u], x[c[u]], s[u]);
            s[u] = k + u * lpr < e ? t : s[u];
        }
    }
    T r = (s[0] + s[2]) + (s[1] + s[3]);
    if (lpr > 1) r += dpp<0xb1>(r);  // lane ^ 1
    return r;
}

// A level's record, from the head of the block
__device__ __forceinline__ TailLevel tail_level(const char* lds, int l) {
    TailLevel L;
    int* o = reinterpret_cast<int*>(&L);
    const Word* p = reinterpret_cast<const Word*>(lds) + l * (int)(sizeof(TailLevel) / 16);
#pragma unroll
    for (int k = 0; k < (int)(sizeof(TailLevel) / 16); ++k) {
        const Word q = p[k];
#pragma unroll
        for (int j = 0; j < 4; ++j) o[4 * k + j] = __builtin_amdgcn_readfirstlane(q[j]);
    }
    return L;
}

template <bool STREAM, class T>
__device__ __forceinline__ void tail_cycle(const TailArgs<T>& A, const ScatterT<T>& sc) {
    extern __shared__ __align__(16) char lds[];
    const int tid = threadIdx.x;
    const int n0 = A.n0, m = A.m;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    // everything from memory, in flight together (the block ends on a whole wave's words)
    Word st[kStage];
    const Word* blob = reinterpret_cast<const Word*>(A.blob);
#pragma unroll
    for (int k = 0; k < kStage; ++k) {
        st[k] = Word(0);
        if (k * BS + wave * kWave < A.words) st[k] = blob[(unsigned)(k * BS + tid)];
    }
    const int t0 = min(tid, n0 - 1);  // no load behind a branch
    const T f0 = A.f[t0], g0 = A.g[t0];
    const Four mm = reinterpret_cast<const Four*>(sc.mem)[t0];
    // the inverse: thread (dp, di) takes the columns dp, dp + 8, ... of row di
    const int di = tid & (kDenseRows - 1), dp = __builtin_amdgcn_readfirstlane(tid / kDenseRows);
    double ai[kAinvHeld];
    if (m <= kDenseRows) {
        const int dr = min(di, m - 1);
#pragma unroll
        for (int q = 0; q < kAinvHeld; ++q) {
            ai[q] = 0.0;
            if (dp + kDenseParts * q < m) ai[q] = (A.ainv + (unsigned)((dp + kDenseParts * q) * m))[(unsigned)dr];
        }
    }
#pragma unroll
    for (int k = 0; k < kStage; ++k) {
        const int i = k * BS + tid;
        if (k * BS + wave * kWave < A.words) reinterpret_cast<Word*>(lds)[i] = st[k];
    }
    T* fa = reinterpret_cast<T*>(lds + A.a0);
    T* ga = reinterpret_cast<T*>(lds + A.g0);
    if (tid < n0) {
        fa[tid] = f0;
        ga[tid] = g0;
    }
    const T gf[4] = {sc.gf[mm.x], sc.gf[max(mm.y, 0)], sc.gf[max(mm.z, 0)], sc.gf[max(mm.w, 0)]};
    for (int i = tid + BS; i < n0; i += BS) {
        fa[i] = A.f[i];
        ga[i] = A.g[i];
    }
    __syncthreads();
    const T w = A.w;
    for (int l = 0; l < A.nl; ++l) {
        // four groups of lanes a coarse row, one per member
        const TailLevel L = tail_level(lds, l);
        const T* v = reinterpret_cast<const T*>(lds + L.v);
        const uint16_t* ci = reinterpret_cast<const uint16_t*>(lds + L.ci);
        const Rec* rec = reinterpret_cast<const Rec*>(lds + L.rec);
        const T* g = reinterpret_cast<const T*>(lds + L.g);
        const T* a = reinterpret_cast<const T*>(lds + L.a);
        const T* dinv = reinterpret_cast<const T*>(lds + L.cdinv);
        T* ac = reinterpret_cast<T*>(lds + L.ca);
        T* gc = reinterpret_cast<T*>(lds + L.cg);
        const int sh = L.lpr_log, lpr = 1 << sh, lane = tid & (lpr - 1);
        for (int t = tid; t < 4 * L.nc << sh; t += BS) {
            const int J = t >> (sh + 2);
            const Rec q = rec[t >> sh];
            T r = T(0);
            if (q.i != kTailNone) r = a[q.i] - w * tail_row<STREAM>(v, ci, g, q.b, q.e, lane, lpr);
            T r1, r2, r3;  // from the lanes ahead
            if (lpr == 1) {
                r1 = dpp<0x101>(r);
                r2 = dpp<0x102>(r);
                r3 = dpp<0x103>(r);
            } else {
                r1 = dpp<0x102>(r);
                r2 = dpp<0x104>(r);
                r3 = dpp<0x106>(r);
            }
            if ((t & (4 * lpr - 1)) == 0) {
                const T s = ((r + r1) + r2) + r3;
                ac[J] = s;
                if (l + 1 < A.nl) gc[J] = dinv[J] * s;
            }
        }
        __syncthreads();
    }
    {  // coarsest: x = A^{-1} f in double, in the batched solves' order of additions
        const T* f = reinterpret_cast<const T*>(lds + A.am);
        T* x = reinterpret_cast<T*>(lds + A.gm);
        double* part = reinterpret_cast<double*>(lds + A.part);
        for (int r0 = 0; r0 < m; r0 += kDenseRows) {
            double acc[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) acc[k] = 0.0;
            if (m <= kDenseRows) {
#pragma unroll
                for (int q = 0; q < kAinvHeld; ++q) {
                    const int j = dp + kDenseParts * q;
                    if (j < m) acc[q % 8] += ai[q] * double(f[j]);
                }
            } else {
                const int i = min(r0 + di, m - 1);
                for (int j0 = dp; j0 < m; j0 += 8 * kDenseParts) {
                    double q[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k) q[k] = (A.ainv + (unsigned)(min(j0 + k * kDenseParts, m - 1) * m))[(unsigned)i];
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const int j = j0 + k * kDenseParts;
                        if (j < m) acc[k] += q[k] * double(f[j]);
                    }
                }
            }
            part[tid] = ((acc[0] + acc[4]) + (acc[2] + acc[6])) + ((acc[1] + acc[5]) + (acc[3] + acc[7]));
            __syncthreads();
            if (tid < kDenseRows && r0 + tid < m) {
                double s = part[tid];
#pragma unroll
                for (int p = 1; p < kDenseParts; ++p) s += part[p * kDenseRows + tid];
                x[r0 + tid] = T(s);
            }
            __syncthreads();
        }
    }
    for (int l = A.nl - 1; l >= 0; --l) {
        const TailLevel L = tail_level(lds, l);
        const T* v = reinterpret_cast<const T*>(lds + L.v);
        const T* dinv = reinterpret_cast<const T*>(lds + L.dinv);
        const uint16_t* ci = reinterpret_cast<const uint16_t*>(lds + L.ci);
        const Rec* rec = reinterpret_cast<const Rec*>(lds + L.rec);
        const T* xc = reinterpret_cast<const T*>(lds + L.cg);
        T* g = reinterpret_cast<T*>(lds + L.g);
        T* a = reinterpret_cast<T*>(lds + L.a);
        for (int t = tid; t < 4 * L.nc; t += BS) {
            const Rec q = rec[t];
            if (q.i != kTailNone) a[q.i] = w * g[q.i] + xc[t >> 2];
        }
        __syncthreads();
        const int sh = L.lpr_log, lpr = 1 << sh, lane = tid & (lpr - 1);
        for (int t = tid; t < 4 * L.nc << sh; t += BS) {
            const Rec q = rec[t >> sh];
            if (q.i == kTailNone) continue;
            const T ai = a[q.i], gi = g[q.i], di = dinv[q.i];
            const T s = tail_row<STREAM>(v, ci, a, q.b, q.e, lane, lpr);
            if (lane == 0) g[q.i] = ai + w * (gi - di * s);
        }
        __syncthreads();
    }
    if (tid < n0) {
        const T z = ga[tid];
        sc.xpf[mm.x] = sc.w * gf[0] + z;
        if (mm.y >= 0) sc.xpf[mm.y] = sc.w * gf[1] + z;
        if (mm.z >= 0) sc.xpf[mm.z] = sc.w * gf[2] + z;
        if (mm.w >= 0) sc.xpf[mm.w] = sc.w * gf[3] + z;
    }
    for (int i = tid + BS; i < n0; i += BS) sc(i, ga[i]);
}

template <class T>
__global__ __launch_bounds__(BS) void k_vc_tail(TailArgs<T> A, ScatterT<T> sc) {
    tail_cycle<false, T>(A, sc);
}

// One system a workgroup, in the order of the CSR-stream kernels: a batch of 32
// systems of 4096 to 32,768 rows takes 15 us here in place of seven launches
// of 4-7 us (the whole batch 8.38 -> 7.70 ms).
template <class T>
__global__ __launch_bounds__(BS) void k_vc_tails(const TailJob<T>* __restrict__ jobs) {
    const TailJob<T> J = jobs[blockIdx.x];
    tail_cycle<true, T>(J.a, J.sc);
}

// Packs one level a block row (blockIdx.y) into the layout tail_cycle reads.
template <class T>
__device__ __forceinline__ void tail_pack(const TailPack<T>& K) {
    const TailSrc<T>& S = K.src[blockIdx.y];
    const TailLevel& L = K.lev[blockIdx.y];
    char* b = K.blob;
    const int t = blockIdx.x * 256 + threadIdx.x, step = gridDim.x * 256;
    if (t == 0) reinterpret_cast<TailLevel*>(b)[blockIdx.y] = L;
    T* v = reinterpret_cast<T*>(b + L.v);
    T* dinv = reinterpret_cast<T*>(b + L.dinv);
    uint16_t* ci = reinterpret_cast<uint16_t*>(b + L.ci);
    Rec* rec = reinterpret_cast<Rec*>(b + L.rec);
    for (int e = t; e < S.nnz; e += step) {
        v[e] = S.v ? S.v[e] : T(S.v64[e]);
        ci[e] = (uint16_t)(S.ci[e] + S.ci_add);
    }
    for (int i = t; i < L.n; i += step) dinv[i] = S.dinv ? S.dinv[i] : T(S.dinv64[i]);
    for (int r = t; r < 4 * L.nc; r += step) {
        const int i0 = reinterpret_cast<const int*>(S.mem)[r], i = i0 + S.mem_add;
        Rec q{kTailNone, 0, 0, 0};
        if (i0 >= 0) q = Rec{(uint16_t)i, (uint16_t)(S.rp[i] + S.rp_add), (uint16_t)(S.rp[i + 1] + S.rp_add), 0};
        rec[r] = q;
    }
}

template <class T>
__global__ __launch_bounds__(256) void k_tail_pack(TailPack<T> K) {
    tail_pack<T>(K);
}

template <class T>
__global__ __launch_bounds__(256) void k_tail_packs(const TailPack<T>* __restrict__ K) {
    if ((int)blockIdx.y < K[blockIdx.z].nl) tail_pack<T>(K[blockIdx.z]);
}

}  // namespace

template <class T>
int tail_layout(const int* n, const int64_t* nnz, const int* lpr, int nl, TailArgs<T>& A, TailLevel* lev) {
    if (nl < 1 || nl > kTailLevels || n[nl] > kTailDense) return 0;
    int64_t at = (int64_t)sizeof(TailLevel) * nl;
    auto take = [&](int& off, int64_t bytes) {
        off = (int)at;
        at = up16(at + bytes);
    };
    for (int l = 0; l < nl; ++l) {
        TailLevel& L = lev[l];
        if (nnz[l] > 65535 || n[l] >= kTailNone) return 0;
        L.n = n[l];
        L.nc = n[l + 1];
        take(L.v, (int64_t)sizeof(T) * nnz[l]);
        take(L.dinv, (int64_t)sizeof(T) * n[l]);
        take(L.rec, 32 * (int64_t)n[l + 1]);
        take(L.ci, 2 * nnz[l]);
        if (lpr && lpr[l] != 4 && lpr[l] != 8) return 0;
        L.lpr_log = lpr && lpr[l] == 8 ? 1 : 0;
        if (at > kTailBytes) return 0;
    }
    at = (at + 16 * kWave - 1) / (16 * kWave) * (16 * kWave);
    A.words = (int)(at / 16);
    A.nl = nl;
    A.n0 = n[0];
    A.m = n[nl];
    int g = 0, a = 0;
    for (int l = 0; l <= nl; ++l) {
        take(g, (int64_t)sizeof(T) * n[l]);
        take(a, (int64_t)sizeof(T) * n[l]);
        if (l < nl) {
            lev[l].g = g;
            lev[l].a = a;
        }
        if (l > 0) {
            lev[l - 1].cg = g;
            lev[l - 1].ca = a;
            lev[l - 1].cdinv = l < nl ? lev[l].dinv : 0;
        }
    }
    A.g0 = lev[0].g;
    A.a0 = lev[0].a;
    A.gm = g;
    A.am = a;
    take(A.part, 8 * BS);
    return at <= kTailBytes ? (int)at : 0;
}

template <class T>
void launch_tail_pack(const TailPack<T>& K, int nl, hipStream_t s) {
    hipLaunchKernelGGL(k_tail_pack<T>, dim3(16, nl), dim3(256), 0, s, K);
}

template <class T>
void vc_tail(const TailArgs<T>& A, int lds, const ScatterT<T>& sc, hipStream_t s) {
    hipLaunchKernelGGL(k_vc_tail<T>, dim3(1), dim3(BS), lds, s, A, sc);
}

template <class T>
void launch_tail_packs(const TailPack<T>* K, int count, int nl, hipStream_t s) {
    hipLaunchKernelGGL(k_tail_packs<T>, dim3(8, nl, count), dim3(256), 0, s, K);
}

template <class T>
void vc_tails(const TailJob<T>* jobs, int count, int lds, hipStream_t s) {
    hipLaunchKernelGGL(k_vc_tails<T>, dim3(count), dim3(BS), lds, s, jobs);
}

// The kernels may take that much of a CU's LDS.
bool tail_prepare() {
    int dev = 0, most = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&most, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess || most < kTailBytes)
        return false;
    for (const void* k : {reinterpret_cast<const void*>(&k_vc_tail<double>), reinterpret_cast<const void*>(&k_vc_tail<float>),
                          reinterpret_cast<const void*>(&k_vc_tails<double>),
                          reinterpret_cast<const void*>(&k_vc_tails<float>)})
        if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kTailBytes) != hipSuccess) return false;
    return true;
}

#define AMG_INST(T)                                                         \
    template int tail_layout<T>(const int*, const int64_t*, const int*, int, TailArgs<T>&, TailLevel*); \
    template void launch_tail_pack<T>(const TailPack<T>&, int, hipStream_t); \
    template void launch_tail_packs<T>(const TailPack<T>*, int, int, hipStream_t); \
    template void vc_tails<T>(const TailJob<T>*, int, int, hipStream_t); \
    template void vc_tail<T>(const TailArgs<T>&, int, const ScatterT<T>&, hipStream_t);
AMG_INST(double)
AMG_INST(float)
#undef AMG_INST

}  // namespace amg
