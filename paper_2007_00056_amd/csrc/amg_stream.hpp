// Row sums of CSR matrices, shared by the level and Krylov kernels: a wave owns
// 64 consecutive rows, a lane one of them.
#pragma once

#include "amg_device.hpp"

namespace amg {

constexpr int kStreamBS = 256;
// entries a wave stages at a time: what its registers hold with enough waves on
// the CU (all of a chunk's loads are in flight together)
template <class T>
constexpr int kWaveChunk = sizeof(T) == 8 ? 512 : 1024;
constexpr int kLongRow = 32;  // entries a row on average: above, rows are long

template <class T>
struct EntAx {  // the entries of A and the x they are applied to
    const T* __restrict__ v;
    const int* __restrict__ ci;
    const T* __restrict__ x;
    __device__ __forceinline__ T at(int i) const { return x[i]; }
};

template <class T>
struct EntDf {  // the same for x = D^{-1} f, formed where it is read
    const T* __restrict__ v;
    const int* __restrict__ ci;
    const double* __restrict__ dinv;
    const double* __restrict__ f;
    __device__ __forceinline__ T at(int i) const { return T(dinv[i] * f[i]); }
};

// ---------------------------------------------------------------------------
// CSR rows.  The entries of a wave's rows are contiguous: they are read with
// coalesced loads, all values and columns of a chunk in flight together and
// then all of its x, and staged in the wave's own part of LDS, from where each
// lane takes its row's.  No barrier, and one chain of three loads a chunk.
//
// ORDER 0: products, rounded, are added in entry order.  ORDER 4 and 8: the
// order of the lane-group kernels with that many lanes a row, one fused sum
// for each lane over every 4th (8th) entry, the sums added as a butterfly adds
// them; such a row is the same bit for bit in either kernel.
//
// Bound by memory on large levels (1.02M rows of 11.5 entries in single
// precision: residual 30.6 us for 106 MB; 33.6 when blocks of 256 rows shared
// the staging with barriers), by the chain of loads on smaller ones.
// ---------------------------------------------------------------------------
template <int K, int ORDER, class T, class Ent>
__device__ __forceinline__ void stage_chunk(const Ent& ent, int c0, int last, T* lds) {
    const int lane = threadIdx.x & (kWave - 1);
    T a[K], x[K];
    int c[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int e = min(c0 + k * kWave + lane, last);
        a[k] = ent.v[e];
        c[k] = ent.ci[e];
    }
#pragma unroll
    for (int k = 0; k < K; ++k) x[k] = ent.at(c[k]);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (ORDER == 0) {
            lds[k * kWave + lane] = a[k] * x[k];
        } else {
            lds[k * kWave + lane] = a[k];
            lds[kWaveChunk<T> + k * kWave + lane] = x[k];
        }
    }
}

// LDS values a wave of the kernel needs
template <class T, int ORDER>
constexpr int kWaveLds = ORDER == 0 ? kWaveChunk<T> : 2 * kWaveChunk<T>;

// Sums of rows row0 .. row0 + 63 below n (a lane each); lds is this wave's.
template <int ORDER = 0, class T, class Ent>
__device__ __forceinline__ T wave_rows(int row0, int n, const int* __restrict__ rp, const Ent& ent, T* lds) {
    static_assert(ORDER == 0 || ORDER == 4 || ORDER == 8, "");
    if (row0 >= n) return T(0);
    const int row = row0 + (int)(threadIdx.x & (kWave - 1));
    const int rb = rp[min(row, n)], re = rp[min(row + 1, n)];
    const int e0 = __builtin_amdgcn_readfirstlane(rb), e1 = __builtin_amdgcn_readlane(re, kWave - 1);
    constexpr int NS = ORDER == 0 ? 1 : ORDER;
    T s[NS];
#pragma unroll
    for (int u = 0; u < NS; ++u) s[u] = T(0);
    for (int c0 = e0; c0 < e1; c0 += kWaveChunk<T>) {
        const int cnt = min(kWaveChunk<T>, e1 - c0), last = c0 + cnt - 1;
        if (cnt <= 5 * kWave) stage_chunk<5, ORDER>(ent, c0, last, lds);
        else if (cnt <= 8 * kWave) stage_chunk<8, ORDER>(ent, c0, last, lds);
        else if constexpr (kWaveChunk<T> > 8 * kWave) {
            if (cnt <= 12 * kWave) stage_chunk<12, ORDER>(ent, c0, last, lds);
            else stage_chunk<16, ORDER>(ent, c0, last, lds);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const int lo = max(rb, c0) - c0, hi = min(re, last + 1) - c0;
        if (ORDER == 0 && e1 - e0 > kLongRow * kWave) {
            // The chunk holds few rows, so a lane's additions are a long chain
            // while the others wait: as few instructions an entry as can be.  With
            // the clamped loads below, SpMV took 105 us on 21,952 rows of 110
            // entries and 172 us on 262,144 of 118 (blocks of 256 rows that share
            // chunks of 2048: 79 and 130); this takes 45 and 91.  At 26 entries the
            // two are equal (34 us on 512,000 rows).
            int e = lo;
            for (; e + 8 <= hi; e += 8) {
                T p[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) p[u] = lds[e + u];
#pragma unroll
                for (int u = 0; u < 8; ++u) s[0] += p[u];
            }
            for (; e < hi; ++e) s[0] += lds[e];
        } else if (ORDER == 0) {
            for (int e = lo; e < hi; e += 4) {
                T p[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) p[u] = lds[min(e + u, hi - 1)];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const T t = s[0] + p[u];
                    s[0] = e + u < hi ? t : s[0];
                }
            }
        } else if (lo < hi) {
            const int b = rb - c0;  // below 0 when the row began in the last chunk
            for (int t = b + (lo - b) / NS * NS; t < hi; t += NS) {
                T a[NS], x[NS];
#pragma unroll
                for (int u = 0; u < NS; ++u) {
                    const int e = min(max(t + u, lo), hi - 1);
                    a[u] = lds[e];
                    x[u] = lds[kWaveChunk<T> + e];
                }
#pragma unroll
                for (int u = 0; u < NS; ++u) {
                    const T q = fma(a[u], x[u], s[u]);
                    s[u] = t + u >= lo && t + u < hi ? q : s[u];
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    if constexpr (ORDER == 8) return ((s[0] + s[4]) + (s[2] + s[6])) + ((s[1] + s[5]) + (s[3] + s[7]));
    else if constexpr (ORDER == 4) return (s[0] + s[2]) + (s[1] + s[3]);
    else return s[0];
}

// Sums of RB consecutive rows from r0 on by a block of RB threads;
// lds: RB / 64 * kWaveLds<T, ORDER> values.
template <class T, int RB = kStreamBS, int ORDER = 0, class Ent>
__device__ __forceinline__ T stream_rows(int r0, int n, const int* __restrict__ rp, const Ent& ent, T* lds) {
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    return wave_rows<ORDER>(r0 + w * kWave, n, rp, ent, lds + w * kWaveLds<T, ORDER>);
}

// ---------------------------------------------------------------------------
// Rows whose columns are coded per slice of 64 rows.
//
// Where neighbouring rows have their entries at the same few distances from
// the diagonal (a matrix of a grid, in any numbering that keeps lines
// together), a slice of 64 rows needs no column per entry: the distinct
// distances col - row of the slice, at most 8, each with the lanes that have
// it.  The values stay where they are.  A row's sum then reads 8 bytes per
// entry instead of 12 (4 instead of 8 with float values) and one 128-byte
// record per 64 rows, its x loads are coalesced and wait for no column, and a
// wave needs no barrier: it copies its slice's values to its own part of LDS
// and each lane takes its row's from there.
//
// Bound by memory.  On 160^3 rows in double (7 entries a row) q = A p with
// (p, q) takes 63 us where the CSR rows took 93 (295 MB, 4.7 TB/s; a copy of
// this size reaches 5.0); on 128^3 rows the residual 25 us (40), the
// postsmoothing 34 (51); with float values on 160^3 the residual 31 us (73)
// and the postsmoothing 45 (79).  Coarse levels that keep the pattern (128^3:
// 524,288 and 131,072 rows) bring a V-cycle there from 174 to 161 us.
//
// The products are added in entry order and not fused with the additions, so
// a row's sum is bit for bit that of stream_rows.  A slice that needs more
// distances is marked (cnt < 0) and read from the CSR arrays, lane by lane.
// ---------------------------------------------------------------------------
constexpr int kCodeSlots = 8;
constexpr int kCodeLevels = 16;  // levels that may have codes
constexpr int kCodeSpare = 64;  // codes are used where at most one slice in so many lacks one

struct alignas(128) SliceCode {
    unsigned long long mask[kCodeSlots];  // lanes whose row has an entry at off[k]
    int off[kCodeSlots];                  // col - row, ascending
    int first;                            // the slice's first entry
    int total, last;                      // its entries; total - 1
    int cnt;                              // distances in use; < 0: not coded
    int pad[4];
};
static_assert(sizeof(SliceCode) == 128, "one cache line");

// The sums of a coded slice with at most K distances, by a wave that has rows of
// it.  Every load is made (an absent entry's, from the row itself), so none
// waits for a branch.
// lds: kCodeSlots * kWave values owned by this wave.
template <int K, class T, class Ent>
__device__ __forceinline__ T coded_sum(const SliceCode& c, int row, int n, const Ent& ent, T* lds) {
#pragma clang fp contract(off)
    const int lane = threadIdx.x & (kWave - 1);
    const T* va = ent.v + c.first;
    T a[K], x[K];
#pragma unroll
    for (int k = 0; k < K; ++k) a[k] = va[coded_val(k * kWave + lane, c.last)];
#pragma unroll
    for (int k = 0; k < K; ++k) x[k] = ent.at(coded_col(row, n, __builtin_amdgcn_inverse_ballot_w64(c.mask[k]), c.off[k]));
    int pos = 0;  // entries of the slice before this lane's row
#pragma unroll
    for (int k = 0; k < K; ++k)
        pos = __builtin_amdgcn_mbcnt_hi((unsigned)(c.mask[k] >> 32),
                                        __builtin_amdgcn_mbcnt_lo((unsigned)c.mask[k], pos));
#pragma unroll
    for (int k = 0; k < K; ++k) lds[k * kWave + lane] = a[k];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    T acc = T(0);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const bool on = __builtin_amdgcn_inverse_ballot_w64(c.mask[k]);
        const T p = lds[pos] * x[k];
        const T s = acc + p;
        acc = on ? s : acc;
        pos += on;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    return acc;
}

// One slice's record: the same for the whole wave and constant for the kernel,
// so it is loaded into scalar registers.
__device__ __forceinline__ SliceCode load_code(const SliceCode* code, int slice) {
    const auto& m = ((const __attribute__((address_space(4))) SliceCode*)code)[slice];
    SliceCode c;
#pragma unroll
    for (int k = 0; k < kCodeSlots; ++k) {
        c.mask[k] = m.mask[k];
        c.off[k] = m.off[k];
    }
    c.first = m.first;
    c.total = m.total;
    c.last = m.last;
    c.cnt = m.cnt;
    return c;
}

// The record has arrived: said where all of it should have, or the compiler
// loads each part where it is first used.
__device__ __forceinline__ void hold_code(SliceCode& c) {
#pragma unroll
    for (int k = 0; k < kCodeSlots; ++k) asm volatile("" : "+s"(c.mask[k]), "+s"(c.off[k]));
    asm volatile("" : "+s"(c.first), "+s"(c.total), "+s"(c.last), "+s"(c.cnt));
}

template <class T, class Ent>
__device__ __forceinline__ T coded_row(const SliceCode& c, int row, int n, const int* __restrict__ rp, const Ent& ent,
                                       T* lds) {
#pragma clang fp contract(off)
    if (c.cnt >= 0) {
        if (c.cnt <= 5) return coded_sum<5>(c, row, n, ent, lds);
        if (c.cnt <= 7) return coded_sum<7>(c, row, n, ent, lds);
        return coded_sum<kCodeSlots>(c, row, n, ent, lds);
    }
    T acc = T(0);
    if (row < n) {
        const int e1 = rp[row + 1];
        for (int e = rp[row]; e < e1; ++e) {
            const T p = ent.v[e] * ent.at(ent.ci[e]);
            acc += p;
        }
    }
    return acc;
}

// What a row kernel reads its matrix rows from: a CSR matrix with the x it is
// applied to, and the codes of its rows when KIND is kCoded; else KIND is the
// order of additions.
constexpr int kCoded = 1;
template <class T, int KIND, class Ent = EntAx<T>>
struct RowSrc {
    // LDS values of a block of RB threads
    template <int RB>
    static constexpr int lds = RB / kWave * (KIND == kCoded ? kCodeSlots * kWave : kWaveLds<T, KIND == kCoded ? 0 : KIND>);
    const SliceCode* code;
    const int* __restrict__ rp;
    Ent ent;
    // For every row of this block of RB threads, RB rows at a time:
    // in = pre(row), what the row's thread reads besides the matrix, loaded
    // ahead of the sum; then body(row, sum, in).  Each XCD takes one contiguous
    // part of the rows, also where its blocks make several steps: x lines that
    // neighbouring rows share are read into one L2.
    template <int RB, class Pre, class Body>
    __device__ __forceinline__ void rows(int n, T* lds, Pre pre, Body body) const {
        const BlockRange mine = xcd_range((n + RB - 1) / RB, blockIdx.x, gridDim.x);
        if constexpr (KIND == kCoded) {
            const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
            SliceCode c = load_code(code, slice_at(wave_slice(mine.first, RB, w), n));
            hold_code(c);
            for (int b = mine.first; b < mine.end; b += mine.step) {
                const int row = b * RB + threadIdx.x;
                const auto in = pre(min(row, n - 1));
                // the next slice's record arrives during this slice's loads
                SliceCode next = load_code(code, slice_at(wave_slice(b + mine.step, RB, w), n));
                T s = T(0);
                if (wave_has_rows(wave_slice(b, RB, w), n)) s = coded_row<T>(c, row, n, rp, ent, lds + w * kCodeSlots * kWave);
                // every load has been used: said here, the loop has no wait for
                // the last slice's store at its head
                __builtin_amdgcn_s_waitcnt(0x0f70);
                hold_code(next);
                if (row < n) body(row, s, in);
                c = next;
            }
        } else {
            for (int b = mine.first; b < mine.end; b += mine.step) {
                const int row = b * RB + threadIdx.x;
                const auto in = pre(min(row, n - 1));
                const T s = stream_rows<T, RB, KIND>(b * RB, n, rp, ent, lds);
                if (row < n) body(row, s, in);
            }
        }
    }
};

inline int stream_blocks(int n, int cap) {
    const int b = (n + kStreamBS - 1) / kStreamBS;
    return b < cap ? (b < 1 ? 1 : b) : cap;
}

}  // namespace amg
