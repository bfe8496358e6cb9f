// Setup-phase kernels: CSR validation and D^{-1}, coarse numbering of a
// matching (Algorithm 2) by prefix sum, the 0/1 Galerkin product P^T A P and
// aggregate member lists.  The matching itself is in k_hem.hip, the coarsest
// level's inverse in k_dense.hip.
#include <climits>
#include <type_traits>

#include "amg_device.hpp"
#include "amg_internal.hpp"
#include "amg_stream.hpp"

namespace amg {

namespace {
constexpr int BS = 256;
inline int blocks_for(int64_t work, int bs = BS, int cap = 1 << 30) {
    int64_t b = (work + bs - 1) / bs;
    if (b < 1) b = 1;
    return (int)(b < cap ? b : cap);
}
}  // namespace

// ---------------------------------------------------------------------------
// Validation of level 0 and inverse diagonal (the Jacobi smoother's D^{-1}).
// Row bounds are checked before any entry of the row is read.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(BS) void k_validate(int n, int64_t nnz, const int* __restrict__ rp,
                                                 const int* __restrict__ ci, const double* __restrict__ v,
                                                 double* __restrict__ dinv, int* err) {
    const int i = blockIdx.x * BS + threadIdx.x;
    if (i >= n) return;
    const int b = rp[i], e = rp[i + 1];
    int bits = 0;
    if (i == 0 && b != 0) bits |= ERR_STRUCT;
    if (i == n - 1 && (int64_t)e != nnz) bits |= ERR_STRUCT;
    if (b < 0 || e < b || (int64_t)e > nnz) {
        atomicOr(err, bits | ERR_STRUCT);
        return;
    }
    double d = 0.0;
    bool has_d = false;
    int prev = -1;
    // no early exit, so the loads of several entries are in flight together
#pragma unroll 4
    for (int k = b; k < e; ++k) {
        const int c = ci[k];
        const double x = v[k];
        if (c < 0 || c >= n || c <= prev) bits |= ERR_STRUCT;
        prev = c;
        if (!isfinite(x)) bits |= ERR_NONFINITE;
        if (c == i) {
            has_d = true;
            d = x;
        }
    }
    if (!has_d || d == 0.0) bits |= ERR_DIAG;
    dinv[i] = has_d && d != 0.0 ? 1.0 / d : 0.0;
    if (bits) atomicOr(err, bits);
}

void launch_validate(int n, int64_t nnz, const int* rp, const int* ci, const double* v, double* dinv, int* err,
                     hipStream_t s) {
    hipLaunchKernelGGL(k_validate, dim3(blocks_for(n)), dim3(BS), 0, s, n, nnz, rp, ci, v, dinv, err);
}

// Column codes: a wave takes a slice of 64 rows, a lane a row, whose distances
// from the diagonal it holds in registers, ascending.  Each step takes the
// smallest distance of the wave and the lanes that have it.  Bound by the
// columns' reads.
__global__ __launch_bounds__(BS) void k_code_slices(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                                                    SliceCode* __restrict__ code, int* __restrict__ uncoded) {
    const int lane = threadIdx.x & (kWave - 1);
    const int slices = (n + kWave - 1) / kWave;
    int bad = 0;
    for (int sl = blockIdx.x * (BS / kWave) + threadIdx.x / kWave; sl < slices; sl += gridDim.x * (BS / kWave)) {
        const int row = sl * kWave + lane;
        const int b = row < n ? rp[row] : 0, len = row < n ? rp[row + 1] - b : 0;
        int d[kCodeSlots];
#pragma unroll
        for (int k = 0; k < kCodeSlots; ++k) d[k] = k < len ? ci[b + k] - row : INT_MAX;
        unsigned long long mask = 0;
        int off = 0, cnt = 0;
#pragma unroll
        for (int k = 0; k < kCodeSlots; ++k) {
            // any lane's distance, then one of the smaller ones while there are any:
            // the lanes of a slice agree on nearly all of them
            int m = INT_MAX;
            for (unsigned long long less; (less = __ballot(d[0] < m)) != 0;)
                m = __builtin_amdgcn_readlane(d[0], __builtin_ctzll(less));
            const bool mine = m != INT_MAX && d[0] == m;
            const unsigned long long who = __ballot(mine);
            if (lane == k) {
                mask = who;
                off = who ? m : 0;
            }
            cnt += who != 0;
#pragma unroll
            for (int j = 0; j + 1 < kCodeSlots; ++j) d[j] = mine ? d[j + 1] : d[j];
            if (mine) d[kCodeSlots - 1] = INT_MAX;
        }
        const bool over = __ballot(len > kCodeSlots || d[0] != INT_MAX) != 0;
        bad += over;
        SliceCode* c = code + sl;
        if (lane < kCodeSlots) {
            c->mask[lane] = mask;
            c->off[lane] = off;
        }
        if (lane == 0) {
            const int last = min(sl * kWave + kWave, n);
            c->first = b;
            c->total = rp[last] - b;
            c->last = rp[last] - b - 1;
            c->cnt = over ? -1 : cnt;
        }
    }
    if (lane == 0 && bad) atomicAdd(uncoded, bad);
}

size_t slice_code_bytes(int n) { return sizeof(SliceCode) * (size_t)((n + kWave - 1) / kWave); }

void launch_code_slices(int n, const int* rp, const int* ci, SliceCode* code, int* uncoded, hipStream_t s) {
    const int nb = blocks_for(n);
    hipLaunchKernelGGL(k_code_slices, dim3(nb < 2048 ? nb : 2048), dim3(BS), 0, s, n, rp, ci, code, uncoded);
}

__global__ __launch_bounds__(BS) void k_dinv(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                                             const double* __restrict__ v, double* __restrict__ dinv, int* err) {
    const int i = blockIdx.x * BS + threadIdx.x;
    if (i >= n) return;
    double d = 0.0;
    for (int k = rp[i]; k < rp[i + 1]; ++k)
        if (ci[k] == i) d = v[k];
    if (d == 0.0 || !isfinite(d)) atomicOr(err, ERR_DIAG);
    dinv[i] = d != 0.0 ? 1.0 / d : 0.0;
}

void launch_dinv(int n, const int* rp, const int* ci, const double* v, double* dinv, int* err, hipStream_t s) {
    hipLaunchKernelGGL(k_dinv, dim3(blocks_for(n)), dim3(BS), 0, s, n, rp, ci, v, dinv, err);
}

// ---------------------------------------------------------------------------
// The two exclusive prefix sums of a pass, with what precedes and follows them
// in the same kernels:
//   numbering   over the leader flags; hands out the coarse ids.  Algorithm 2
//               does so when the smaller vertex of a pair (or a singleton) is
//               visited: ids are ranks of the aggregates' minimum vertex.
//   row offsets over the coarse rows' entry counts; hands the host its words.
// Up to ONE_MAX items one workgroup does all of it in one launch (9 us at
// 14,000 rows, 4 up to 4096, where flags, three scan phases and assignment took
// five kernels of 3-5 us each); above, three phases: tile sums, scan of the
// tile sums, apply.
// ---------------------------------------------------------------------------
namespace {
constexpr int SCAN_ITEMS = 8;
constexpr int SCAN_TILE = BS * SCAN_ITEMS;
constexpr int ONE_BS = 1024;
constexpr int ONE_TILES = 4;
constexpr int ONE_MAX = ONE_TILES * 4 * ONE_BS;

__device__ __forceinline__ int block_excl_scan(int x, int& total) {
    __shared__ int sh[BS / kWave];
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    int inc = x;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int y = __shfl_up(inc, off, kWave);
        if (lane >= off) inc += y;
    }
    if (lane == kWave - 1) sh[wid] = inc;
    __syncthreads();
    int pre = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < BS / kWave; ++w) {
        const int t = sh[w];
        if (w < wid) pre += t;
        total += t;
    }
    __syncthreads();
    return pre + inc - x;
}

// Numbering: item v is 1 where v leads its aggregate.
struct Numbering {
    const int* __restrict__ mate;
    int* __restrict__ agg;
    int* __restrict__ lead;
    int* __restrict__ total;  // coarse rows
    int* novf;                // cleared for the Galerkin product
    __device__ __forceinline__ int load(int v) const { return mate[v]; }
    __device__ __forceinline__ int value(int v, int m) const { return m < 0 || v < m; }
    __device__ __forceinline__ void put(int v, int m, int id) const {
        if (m >= 0 && m < v) return;
        agg[v] = id;
        if (m >= 0) agg[m] = id;
        lead[id] = v;
    }
    // by one wave of one block, once the total is known
    __device__ __forceinline__ void finish(int n, int sum) const {
        if (threadIdx.x != 0) return;
        *total = sum;
        *novf = 0;
    }
};

// Row offsets, and the words a pass hands to the host (mapped memory): the
// matching's 8 counters, cleared for the next pass, the coarse row count, the
// coarse entry count, the error word and the Galerkin product's overflow rows;
// then seq (system scope).
struct Offsets {
    const int* __restrict__ cnt;
    int* __restrict__ crp;
    PassWords w;
    __device__ __forceinline__ int load(int i) const { return cnt[i]; }
    __device__ __forceinline__ int value(int, int c) const { return c; }
    __device__ __forceinline__ void put(int i, int, int at) const { crp[i] = at; }
    __device__ __forceinline__ void finish(int n, int sum) const {
        const int t = threadIdx.x;
        if (t >= kWave) return;
        if (t < 8) {
            w.out[t] = w.cnt[t];
            w.cnt[t] = 0;
        } else if (t == 8) {
            w.out[8] = *w.nc;
        } else if (t == 9) {
            w.out[9] = sum;
            crp[n] = sum;
        } else if (t == 10) {
            w.out[10] = *w.err;
        } else if (t == 11) {
            w.out[11] = *w.novf;
        }
        __threadfence_system();  // the wave's words before the sequence word
        if (t == 0) __hip_atomic_store(&w.out[kPassSeq], w.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
};
}  // namespace

// One workgroup: a thread holds 4 neighbouring items of each of T tiles.
template <int T, class Op>
__global__ __launch_bounds__(ONE_BS) void k_scan_one(int n, Op op) {
    constexpr int NW = ONE_BS / kWave;
    __shared__ int sums[T * NW];
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    int raw[T][4], pre[T];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) raw[t][j] = op.load(min((t * ONE_BS + (int)threadIdx.x) * 4 + j, n - 1));
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const int i = (t * ONE_BS + threadIdx.x) * 4;
        int x = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) x += i + j < n ? op.value(i + j, raw[t][j]) : 0;
        int inc = x;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const int y = __shfl_up(inc, off, kWave);
            if (lane >= off) inc += y;
        }
        if (lane == kWave - 1) sums[t * NW + wid] = inc;
        pre[t] = inc - x;
    }
    __syncthreads();
    static_assert(T * NW <= kWave, "a sum a lane");
    // every wave scans the waves' sums for itself
    const int own = lane < T * NW ? sums[lane] : 0;
    int inc = own;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int y = __shfl_up(inc, off, kWave);
        if (lane >= off) inc += y;
    }
    const int total = __shfl(inc, kWave - 1, kWave);
#pragma unroll
    for (int t = 0; t < T; ++t) {
        int ex = pre[t] + __shfl(inc - own, t * NW + wid, kWave);
        const int i = (t * ONE_BS + threadIdx.x) * 4;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (i + j >= n) continue;
            op.put(i + j, raw[t][j], ex);
            ex += op.value(i + j, raw[t][j]);
        }
    }
    op.finish(n, total);
}

template <class Op>
__global__ __launch_bounds__(BS) void k_scan_tiles(int n, Op op, int* __restrict__ tsum) {
    const int base = blockIdx.x * SCAN_TILE + threadIdx.x * SCAN_ITEMS;
    int s = 0;
#pragma unroll
    for (int t = 0; t < SCAN_ITEMS; ++t)
        if (base + t < n) s += op.value(base + t, op.load(base + t));
    int total;
    block_excl_scan(s, total);
    if (threadIdx.x == 0) tsum[blockIdx.x] = total;
}

__global__ __launch_bounds__(BS) void k_scan_top(int* tsum, int nt) {
    int carry = 0;
    for (int base = 0; base < nt; base += BS) {
        const int i = base + threadIdx.x;
        const int x = i < nt ? tsum[i] : 0;
        int total;
        const int ex = block_excl_scan(x, total);
        if (i < nt) tsum[i] = carry + ex;
        carry += total;
    }
    if (threadIdx.x == 0) tsum[nt] = carry;
}

template <class Op>
__global__ __launch_bounds__(BS) void k_scan_apply(int n, Op op, const int* __restrict__ tsum, int nt) {
    const int base = blockIdx.x * SCAN_TILE + threadIdx.x * SCAN_ITEMS;
    int raw[SCAN_ITEMS];
    int s = 0;
#pragma unroll
    for (int t = 0; t < SCAN_ITEMS; ++t) {
        raw[t] = op.load(min(base + t, n - 1));
        s += base + t < n ? op.value(base + t, raw[t]) : 0;
    }
    int total;
    int ex = block_excl_scan(s, total) + tsum[blockIdx.x];
#pragma unroll
    for (int t = 0; t < SCAN_ITEMS; ++t) {
        if (base + t >= n) continue;
        op.put(base + t, raw[t], ex);
        ex += op.value(base + t, raw[t]);
    }
    if (blockIdx.x == 0) op.finish(n, tsum[nt]);
}

size_t scan_tmp_ints(int n) { return (size_t)(n + SCAN_TILE - 1) / SCAN_TILE + 1; }

template <class Op>
static void scan_launch(int n, const Op& op, int* tmp, hipStream_t s) {
    if (n <= 4 * ONE_BS) {
        hipLaunchKernelGGL((k_scan_one<1, Op>), dim3(1), dim3(ONE_BS), 0, s, n, op);
    } else if (n <= ONE_MAX) {
        hipLaunchKernelGGL((k_scan_one<ONE_TILES, Op>), dim3(1), dim3(ONE_BS), 0, s, n, op);
    } else {
        const int nt = (n + SCAN_TILE - 1) / SCAN_TILE;
        hipLaunchKernelGGL(k_scan_tiles<Op>, dim3(nt), dim3(BS), 0, s, n, op, tmp);
        hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(BS), 0, s, tmp, nt);
        hipLaunchKernelGGL(k_scan_apply<Op>, dim3(nt), dim3(BS), 0, s, n, op, tmp, nt);
    }
}

void launch_numbering(int n, const int* mate, int* agg, int* lead, int* nc, int* novf, int* tmp, hipStream_t s) {
    scan_launch(n, Numbering{mate, agg, lead, nc, novf}, tmp, s);
}

void launch_offsets(int n, const int* rowcnt, int* crp, const PassWords& w, int* tmp, hipStream_t s) {
    scan_launch(n, Offsets{rowcnt, crp, w}, tmp, s);
}

// ---------------------------------------------------------------------------
// Galerkin product of one matching pass, A_c = P^T B P with P_{i,agg(i)} = 1
// (Section 2.1.1).  Coarse row I has members lead[I] < mate[lead[I]]; entry
// (I,J) sums b_ij over the members in ascending order and, within a member,
// over its columns in ascending order, the first term initialising the sum.
// The fixed order makes the values bit-identical on every run.
//
// G lanes (16 or 32) take a coarse row, a lane one entry of its members, or
// two.  The entries' coarse columns go through LDS, where each lane compares
// its own with all of the row's: the bits of the equal and of the smaller ones.
// An entry with no equal one before it leads its column, whose rank is the
// number of smaller leaders, and adds the values of the equal ones in order.
// Rows of more than 2 G entries go to a slower path.
//
// Bound by the chain of loads up to the coarse columns and, on large levels,
// by the comparisons.  A thread a coarse row, inserting into a sorted list in
// LDS, took 40-50 us to count and 50-60 to fill on any small level of 15-30
// entries a row; this takes 5-8 and 7-15.  On 27,700 rows of 17 entries
// 41 + 51 us became 11 + 18, on 218,000 of 12 23 + 51 became 19 + 29; on 2.1M
// rows of 7 38 + 129 became 73 + 119.
// ---------------------------------------------------------------------------
namespace {
constexpr int RAP_BS = 256;
constexpr int RAP_MAX = 4096;  // blocks: two rounds of the chip
inline int rap_lanes(int n, int64_t nnz) { return nnz <= 8 * (int64_t)n ? 16 : 32; }

// The row's L <= G * E entries from b0 on (l0 of them) and from b1 on; key and
// val are the row's places in LDS.  Returns the distinct columns.
template <int G, int E, bool FILL>
__device__ __forceinline__ int rap_row(int l0, int b0, int b1, int L, const int* __restrict__ ci,
                                       const double* __restrict__ v, const int* __restrict__ agg, int* key,
                                       double* val, int o, int* __restrict__ cci, double* __restrict__ cv) {
    using Bits = std::conditional_t<(G * E > 32), unsigned long long, unsigned>;
    const int lane = threadIdx.x & (G - 1), base = threadIdx.x & (kWave - 1) & ~(G - 1);
    int c[E], J[E];
    double x[E];
#pragma unroll
    for (int t = 0; t < E; ++t) {
        const int k = lane + G * t, e = k < l0 ? b0 + k : b1 + (k - l0);
        c[t] = k < L ? ci[e] : -1;
        x[t] = FILL && k < L ? v[e] : 0.0;
    }
#pragma unroll
    for (int t = 0; t < E; ++t) J[t] = c[t] >= 0 ? agg[c[t]] : INT_MAX;
#pragma unroll
    for (int t = 0; t < E; ++t) {
        key[lane + G * t] = J[t];
        if (FILL) val[lane + G * t] = x[t];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    Bits eq[E], lt[E];
#pragma unroll
    for (int t = 0; t < E; ++t) eq[t] = lt[t] = 0;
    for (int j = 0; j < L; j += 4) {
        const int4 q = *reinterpret_cast<const int4*>(key + j);
#pragma unroll
        for (int t = 0; t < E; ++t) {
            eq[t] |= Bits((q.x == J[t]) | (q.y == J[t]) << 1 | (q.z == J[t]) << 2 | (q.w == J[t]) << 3) << j;
            lt[t] |= Bits((q.x < J[t]) | (q.y < J[t]) << 1 | (q.z < J[t]) << 2 | (q.w < J[t]) << 3) << j;
        }
    }
    Bits leaders = 0;
    bool lead[E];
#pragma unroll
    for (int t = 0; t < E; ++t) {
        const int k = lane + G * t;
        lead[t] = k < L && (eq[t] & ((Bits(1) << k) - 1)) == 0;
        const unsigned b = unsigned(__ballot(lead[t]) >> base) & unsigned((1ull << G) - 1);
        leaders |= Bits(b) << (G * t);
    }
    const int count = sizeof(Bits) == 8 ? __popcll(leaders) : __popc(unsigned(leaders));
    if (FILL) {
#pragma unroll
        for (int t = 0; t < E; ++t) {
            if (!lead[t]) continue;
            double sum = x[t];
            for (Bits m = eq[t] & (eq[t] - 1); m != 0; m &= m - 1)
                sum += val[sizeof(Bits) == 8 ? __builtin_ctzll(m) : __builtin_ctz(unsigned(m))];
            const Bits below = lt[t] & leaders;
            const int r = o + (sizeof(Bits) == 8 ? __popcll(below) : __popc(unsigned(below)));
            cci[r] = J[t];
            cv[r] = sum;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    return count;
}
}  // namespace

// FILL: rows below nmax get their columns and values from crp on.  Else they
// are counted up to nmax (an upper bound of the coarse size *ncp); rows past
// the coarse size count zero, so a scan over nmax rows gives the offsets.
template <int G, bool FILL>
__global__ __launch_bounds__(RAP_BS) void k_rap(int nmax, const int* __restrict__ ncp, const int* __restrict__ lead,
                                                const int* __restrict__ mate, const int* __restrict__ rp,
                                                const int* __restrict__ ci, const double* __restrict__ v,
                                                const int* __restrict__ agg, int* __restrict__ rowcnt,
                                                int* __restrict__ ovf, int* novf, const int* __restrict__ crp,
                                                int* __restrict__ cci, double* __restrict__ cv) {
    __shared__ __align__(16) int skey[2 * RAP_BS];
    __shared__ double sval[FILL ? 2 * RAP_BS : 1];
    const int g = threadIdx.x / G, lane = threadIdx.x & (G - 1);
    int* key = skey + g * 2 * G;
    double* val = sval + (FILL ? g * 2 * G : 0);
    const int nc = FILL ? nmax : *ncp;
    for (int I = blockIdx.x * (RAP_BS / G) + g; I < nc; I += gridDim.x * (RAP_BS / G)) {
        const int m0 = lead[I];
        const int m1 = mate[m0];
        const int b0 = rp[m0], l0 = rp[m0 + 1] - b0;
        const int b1 = m1 >= 0 ? rp[m1] : 0, L = l0 + (m1 >= 0 ? rp[m1 + 1] - b1 : 0);
        int cnt = 0;
        if (L > 2 * G) {  // the slow path's
            if (!FILL && lane == 0) ovf[atomicAdd(novf, 1)] = I;
        } else {
            const int o = FILL ? crp[I] : 0;
            cnt = L <= G ? rap_row<G, 1, FILL>(l0, b0, b1, L, ci, v, agg, key, val, o, cci, cv)
                         : rap_row<G, 2, FILL>(l0, b0, b1, L, ci, v, agg, key, val, o, cci, cv);
        }
        if (!FILL && lane == 0) rowcnt[I] = cnt;
    }
    if (!FILL)
        for (int I = nc + blockIdx.x * RAP_BS + threadIdx.x; I < nmax; I += gridDim.x * RAP_BS) rowcnt[I] = 0;
}

// Overflow rows (more than two entries a lane): one wave per
// row.  The row's entries, in member-then-column order, are staged in LDS
// with their coarse columns; a stable rank (by column, then entry order)
// sorts them, and the first lane of each run of equal columns adds the run
// in entry order, so the sums are the same as on the fast path.  Rows longer
// than RAP_SLOW_CAP entries fall back to one lane working in place.
namespace {
constexpr int RAP_SLOW_CAP = 1024;

__device__ __forceinline__ int rap_entry(int k, int l0, int b0, int b1) { return k < l0 ? b0 + k : b1 + (k - l0); }

// serial fallback: distinct columns of a long row
__device__ int rap_count_serial(const int mm[2], const int* __restrict__ rp, const int* __restrict__ ci,
                                const int* __restrict__ agg) {
    int count = 0;
    for (int a = 0; a < 2; ++a) {
        if (mm[a] < 0) continue;
        for (int e = rp[mm[a]]; e < rp[mm[a] + 1]; ++e) {
            const int J = agg[ci[e]];
            bool seen = false;
            for (int b = 0; b <= a && !seen; ++b) {
                if (mm[b] < 0) continue;
                const int end = (b == a) ? e : rp[mm[b] + 1];
                for (int f = rp[mm[b]]; f < end; ++f)
                    if (agg[ci[f]] == J) {
                        seen = true;
                        break;
                    }
            }
            count += !seen;
        }
    }
    return count;
}

// serial fallback: sorted insertion into the row's own output segment
__device__ void rap_fill_serial(const int mm[2], const int* __restrict__ rp, const int* __restrict__ ci,
                                const double* __restrict__ v, const int* __restrict__ agg, int o,
                                int* __restrict__ cci, double* __restrict__ cv) {
    int len = 0;
    for (int a = 0; a < 2; ++a) {
        if (mm[a] < 0) continue;
        for (int e = rp[mm[a]]; e < rp[mm[a] + 1]; ++e) {
            const int J = agg[ci[e]];
            int lo = 0, hi = len;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (cci[o + mid] < J) lo = mid + 1;
                else hi = mid;
            }
            if (lo < len && cci[o + lo] == J) {
                cv[o + lo] += v[e];
            } else {
                for (int q = len; q > lo; --q) {
                    cci[o + q] = cci[o + q - 1];
                    cv[o + q] = cv[o + q - 1];
                }
                cci[o + lo] = J;
                cv[o + lo] = v[e];
                ++len;
            }
        }
    }
}
}  // namespace

template <bool FILL>
__global__ __launch_bounds__(kWave) void k_rap_slow(const int* __restrict__ ovf, const int* novf,
                                                    const int* __restrict__ lead, const int* __restrict__ mate,
                                                    const int* __restrict__ rp, const int* __restrict__ ci,
                                                    const double* __restrict__ v, const int* __restrict__ agg,
                                                    int* __restrict__ rowcnt, const int* __restrict__ crp,
                                                    int* __restrict__ cci, double* __restrict__ cv) {
    __shared__ int key[RAP_SLOW_CAP], skey[RAP_SLOW_CAP];
    __shared__ double val[RAP_SLOW_CAP], sval[RAP_SLOW_CAP];
    __shared__ int s_cnt;
    const int lane = threadIdx.x;
    const int nrows = *novf;
    for (int t = blockIdx.x; t < nrows; t += gridDim.x) {
        const int I = ovf[t];
        const int m0 = lead[I];
        const int mm[2] = {m0, mate[m0]};
        const int b0 = rp[m0], l0 = rp[m0 + 1] - b0;
        const int b1 = mm[1] >= 0 ? rp[mm[1]] : 0, l1 = mm[1] >= 0 ? rp[mm[1] + 1] - b1 : 0;
        const int L = l0 + l1;
        if (L > RAP_SLOW_CAP) {
            if (lane == 0) {
                if (FILL) rap_fill_serial(mm, rp, ci, v, agg, crp[I], cci, cv);
                else rowcnt[I] = rap_count_serial(mm, rp, ci, agg);
            }
            continue;
        }
        if (lane == 0) s_cnt = 0;
        for (int k = lane; k < L; k += kWave) {
            const int e = rap_entry(k, l0, b0, b1);
            key[k] = agg[ci[e]];
            if (FILL) val[k] = v[e];
        }
        __syncthreads();
        int distinct = 0;
        for (int k = lane; k < L; k += kWave) {
            const int J = key[k];
            int less = 0, before = 0;
            for (int j = 0; j < L; ++j) {
                const int K = key[j];
                less += K < J;
                before += (K == J) & (j < k);
            }
            distinct += before == 0;
            if (FILL) {
                skey[less + before] = J;
                sval[less + before] = val[k];
            }
        }
        if (!FILL) {
            if (distinct) atomicAdd(&s_cnt, distinct);
            __syncthreads();
            if (lane == 0) rowcnt[I] = s_cnt;
            __syncthreads();
            continue;
        }
        __syncthreads();
        const int o = crp[I];
        for (int p = lane; p < L; p += kWave) {
            const int J = skey[p];
            if (p > 0 && skey[p - 1] == J) continue;  // not the start of a run
            int d = 0;  // runs before this one = distinct columns below J
            for (int q = 0; q < p; ++q) d += (q == 0 || skey[q - 1] != skey[q]);
            double sum = sval[p];
            for (int q = p + 1; q < L && skey[q] == J; ++q) sum += sval[q];
            cci[o + d] = J;
            cv[o + d] = sum;
        }
        __syncthreads();
    }
}

void launch_rap_count(int nmax, int64_t nnz, const int* ncp, const int* lead, const int* mate, const int* rp,
                      const int* ci, const int* agg, int* rowcnt, int* ovf, int* novf, hipStream_t s) {
    const int G = rap_lanes(nmax, nnz);
    const dim3 g(blocks_for(nmax, RAP_BS / G, RAP_MAX));
    if (G == 16)
        hipLaunchKernelGGL((k_rap<16, false>), g, dim3(RAP_BS), 0, s, nmax, ncp, lead, mate, rp, ci, nullptr, agg,
                           rowcnt, ovf, novf, nullptr, nullptr, nullptr);
    else
        hipLaunchKernelGGL((k_rap<32, false>), g, dim3(RAP_BS), 0, s, nmax, ncp, lead, mate, rp, ci, nullptr, agg,
                           rowcnt, ovf, novf, nullptr, nullptr, nullptr);
}

void launch_rap_count_slow(int nc, const int* ovf, const int* novf, const int* lead, const int* mate, const int* rp,
                           const int* ci, const int* agg, int* rowcnt, hipStream_t s) {
    hipLaunchKernelGGL(k_rap_slow<false>, dim3(blocks_for(nc, 1, 512)), dim3(kWave), 0, s, ovf, novf, lead, mate, rp,
                       ci, nullptr, agg, rowcnt, nullptr, nullptr, nullptr);
}

void launch_rap_fill(int nc, int n, int64_t nnz, const int* lead, const int* mate, const int* rp, const int* ci,
                     const double* v, const int* agg, const int* crp, int* cci, double* cv, hipStream_t s) {
    const int G = rap_lanes(n, nnz);  // the rows left out are those the count left out
    const dim3 g(blocks_for(nc, RAP_BS / G, RAP_MAX));
    if (G == 16)
        hipLaunchKernelGGL((k_rap<16, true>), g, dim3(RAP_BS), 0, s, nc, nullptr, lead, mate, rp, ci, v, agg, nullptr,
                           nullptr, nullptr, crp, cci, cv);
    else
        hipLaunchKernelGGL((k_rap<32, true>), g, dim3(RAP_BS), 0, s, nc, nullptr, lead, mate, rp, ci, v, agg, nullptr,
                           nullptr, nullptr, crp, cci, cv);
}

void launch_rap_fill_slow(int nc, const int* ovf, const int* novf, const int* lead, const int* mate, const int* rp,
                          const int* ci, const double* v, const int* agg, const int* crp, int* cci, double* cv,
                          hipStream_t s) {
    hipLaunchKernelGGL(k_rap_slow<true>, dim3(blocks_for(nc, 1, 512)), dim3(kWave), 0, s, ovf, novf, lead, mate, rp,
                       ci, v, agg, nullptr, crp, cci, cv);
}

// ---------------------------------------------------------------------------
// Level maps: composed aggregate map and member lists of the coarse rows.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(BS) void k_compose(int n, const int* __restrict__ a1, const int* __restrict__ a2,
                                                int* __restrict__ out) {
    const int i = blockIdx.x * BS + threadIdx.x;
    if (i < n) out[i] = a2[a1[i]];
}

void launch_compose(int n, const int* agg1, const int* agg2, int* out, hipStream_t s) {
    hipLaunchKernelGGL(k_compose, dim3(blocks_for(n)), dim3(BS), 0, s, n, agg1, agg2, out);
}

__device__ __forceinline__ void cswap(int& a, int& b) {
    const int lo = a < b ? a : b, hi = a < b ? b : a;
    a = lo;
    b = hi;
}

// lead2 == nullptr: a level made of a single pass (members of pass-1 pairs).
__global__ __launch_bounds__(BS) void k_members(int nc, const int* __restrict__ lead2, const int* __restrict__ mate2,
                                                const int* __restrict__ lead1, const int* __restrict__ mate1,
                                                int4* __restrict__ mem) {
    const int J = blockIdx.x * BS + threadIdx.x;
    if (J >= nc) return;
    constexpr int BIG = 0x7fffffff;
    int m[4] = {BIG, BIG, BIG, BIG};
    if (lead2 == nullptr) {
        const int a = lead1[J], b = mate1[a];
        m[0] = a;
        m[1] = b < 0 ? BIG : b;
    } else {
        const int I1 = lead2[J], I2 = mate2[I1];
        const int a1 = lead1[I1], b1 = mate1[a1];
        m[0] = a1;
        m[1] = b1 < 0 ? BIG : b1;
        if (I2 >= 0) {
            const int a2 = lead1[I2], b2 = mate1[a2];
            m[2] = a2;
            m[3] = b2 < 0 ? BIG : b2;
        }
    }
    cswap(m[0], m[1]);
    cswap(m[2], m[3]);
    cswap(m[0], m[2]);
    cswap(m[1], m[3]);
    cswap(m[1], m[2]);
    int4 o;
    o.x = m[0] == BIG ? -1 : m[0];
    o.y = m[1] == BIG ? -1 : m[1];
    o.z = m[2] == BIG ? -1 : m[2];
    o.w = m[3] == BIG ? -1 : m[3];
    mem[J] = o;
}

void launch_members(int nc, const int* lead2, const int* mate2, const int* lead1, const int* mate1, int4* mem,
                    hipStream_t s) {
    hipLaunchKernelGGL(k_members, dim3(blocks_for(nc)), dim3(BS), 0, s, nc, lead2, mate2, lead1, mate1, mem);
}

// Start of each system inside a concatenated level and its coarse level:
// out[2j] = agg[off[j]] (first coarse row), out[2j+1] = crp[out[2j]].
__global__ __launch_bounds__(BS) void k_seg_starts(int m, const int* __restrict__ off, const int* __restrict__ agg,
                                                   const int* __restrict__ crp, int* __restrict__ out) {
    const int j = blockIdx.x * BS + threadIdx.x;
    if (j >= m) return;
    const int c = agg[off[j]];
    out[2 * j] = c;
    out[2 * j + 1] = crp[c];
}

void launch_seg_starts(int m, const int* off, const int* agg, const int* crp, int* out, hipStream_t s) {
    hipLaunchKernelGGL(k_seg_starts, dim3(blocks_for(m)), dim3(BS), 0, s, m, off, agg, crp, out);
}

}  // namespace amg
