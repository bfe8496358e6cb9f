// CSR-stream building block shared by the level and Krylov kernels.
//
// A block of RB threads (256 by default) owns RB consecutive rows.  It reads their contiguous
// entry range with coalesced, independent loads (values, columns and the
// gathered vector), stages the products in LDS, and then each thread adds
// its own row's products in entry order.  Entries are processed in LDS chunks,
// so rows of any length are handled.
#pragma once

#include "amg_device.hpp"

namespace amg {

constexpr int kStreamBS = 256;
constexpr int kStreamChunk = 2048;  // products per LDS chunk

template <class T>
struct EntAx {  // a_ij x_j
    const T* __restrict__ v;
    const int* __restrict__ ci;
    const T* __restrict__ x;
    __device__ __forceinline__ T operator()(int e) const { return v[e] * x[ci[e]]; }
};

// RB rows per block (the block has RB threads); a row's sum does not depend
// on RB.
template <class T, int RB = kStreamBS, class Ent>
__device__ __forceinline__ T stream_rows(int r0, int n, const int* __restrict__ rp, const Ent& ent, T* prod) {
    constexpr int BS = RB;
    const int r1 = min(r0 + BS, n);
    const int e0 = rp[r0], e1 = rp[r1];
    const int row = r0 + threadIdx.x;
    const int rb = row < r1 ? rp[row] : 0, re = row < r1 ? rp[row + 1] : 0;
    T acc = T(0);
    for (int c0 = e0; c0 < e1; c0 += kStreamChunk) {
        const int c1 = min(c0 + kStreamChunk, e1);
#pragma unroll 4
        for (int e = c0 + threadIdx.x; e < c1; e += BS) prod[e - c0] = ent(e);
        __syncthreads();
        const int lo = max(rb, c0), hi = min(re, c1);
        for (int e = lo; e < hi; ++e) acc += prod[e - c0];
        __syncthreads();
    }
    return acc;
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
// and the postsmoothing 45 (79).
//
// The products are added in entry order and not fused with the additions, so
// a row's sum is bit for bit that of stream_rows.  A slice that needs more
// distances is marked (cnt < 0) and read from the CSR arrays, lane by lane.
// ---------------------------------------------------------------------------
constexpr int kCodeSlots = 8;
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

// The sums of a coded slice with at most K distances.  Every load is made
// (an absent entry's, from the row itself), so none waits for a branch.
// lds: kCodeSlots * kWave values owned by this wave.
template <int K, class T>
__device__ __forceinline__ T coded_sum(const SliceCode& c, int row, int n, const EntAx<T>& ent, T* lds) {
#pragma clang fp contract(off)
    const int lane = threadIdx.x & (kWave - 1);
    const int r = min(row, n - 1);
    const T* va = ent.v + c.first;
    T a[K], x[K];
#pragma unroll
    for (int k = 0; k < K; ++k) a[k] = va[min(k * kWave + lane, c.last)];
#pragma unroll
    for (int k = 0; k < K; ++k) x[k] = ent.x[r + (__builtin_amdgcn_inverse_ballot_w64(c.mask[k]) ? c.off[k] : 0)];
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

template <class T>
__device__ __forceinline__ T coded_row(const SliceCode& c, int row, int n, const int* __restrict__ rp,
                                       const EntAx<T>& ent, T* lds) {
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
            const T p = ent(e);
            acc += p;
        }
    }
    return acc;
}

// What a row kernel reads its matrix rows from: a CSR matrix with the x it is
// applied to, and the codes of its rows when CODED.
template <class T, bool CODED>
struct RowSrc {
    const SliceCode* code;
    const int* __restrict__ rp;
    EntAx<T> ent;
    // For every row of this block of RB threads, RB rows at a time:
    // in = pre(row), what the row's thread reads besides the matrix, loaded
    // ahead of the sum; then body(row, sum, in).  Each XCD takes one contiguous
    // part of the rows, also where its blocks make several steps: x lines that
    // neighbouring rows share are read into one L2.
    template <int RB, class Pre, class Body>
    __device__ __forceinline__ void rows(int n, T* prod, Pre pre, Body body) const {
        const int nb = (n + RB - 1) / RB;
        const int xcd = blockIdx.x % kNumXcd, per = nb / kNumXcd, rem = nb % kNumXcd;
        const int end = (xcd + 1) * per + min(xcd + 1, rem);
        const int step = gridDim.x / kNumXcd + (xcd < (int)gridDim.x % kNumXcd);  // blocks on this XCD
        int b = xcd * per + min(xcd, rem) + blockIdx.x / kNumXcd;
        if constexpr (CODED) {
            static_assert(RB * kCodeSlots <= kStreamChunk, "a wave's part of prod");
            const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
            const int last = (n - 1) / kWave;
            SliceCode c = load_code(code, min(b * (RB / kWave) + w, last));
            hold_code(c);
            for (; b < end; b += step) {
                const int row = b * RB + threadIdx.x;
                const auto in = pre(min(row, n - 1));
                // the next slice's record arrives during this slice's loads
                SliceCode next = load_code(code, min((b + step) * (RB / kWave) + w, last));
                const T s = coded_row<T>(c, row, n, rp, ent, prod + w * kCodeSlots * kWave);
                // every load has been used: said here, the loop has no wait for
                // the last slice's store at its head
                __builtin_amdgcn_s_waitcnt(0x0f70);
                hold_code(next);
                if (row < n) body(row, s, in);
                c = next;
            }
        } else {
            for (; b < end; b += step) {
                const int row = b * RB + threadIdx.x;
                const auto in = pre(min(row, n - 1));
                const T s = stream_rows<T, RB>(b * RB, n, rp, ent, prod);
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
