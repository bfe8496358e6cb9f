// Node-based heavy edge matching (Section 2.1.1, Algorithm 2) on the GPU.
//
// Algorithm 2 visits the vertices in ascending order; an unmatched vertex v
// takes its heaviest unmatched higher neighbour (lowest index on ties; the
// lower ones are matched, or were left alone, by then).  Whether edge v -> w
// (v < w) is taken depends on lower vertices alone:
//
//   avail(w, v)  no edge x -> w with x < v is taken
//   take(v -> w) no edge x -> v is taken, avail(w, v), and no neighbour that
//                v prefers to w is available to v
//
// Each vertex keeps one word: bit k says that its k-th lower edge (in column
// order) is known not to be taken ("dead"); the top bit says that one is
// taken, and then every other bit is set, so the zero bit names the taker.
// avail(w, v) holds once the bits below v's position in w's word are all set,
// and fails once the top bit is set without that.  v walks its preference
// list: an unavailable choice is skipped; an available one makes all later
// edges of v dead at once (whatever becomes of v); and once all of v's own
// lower edges are dead, v takes it.  A taken vertex makes all its edges dead.
//
// Bits are only ever set, and each is a fact of the one greedy matching, so
// a stale word only delays: no rounds, no barriers and no order between
// words are needed, and the result is Algorithm 2's, bit for bit, whatever
// the timing.  The lowest undecided vertex can always decide, so the walk ends.
//
// That holds as long as no conclusion rests on a bit being absent from one word
// when it was set before a bit seen in another.  "Unavailable" is such a
// conclusion: a top bit without the lower ones.  Where these share a word, one
// read has both.  In a vertex with more lower edges than a word holds they are
// in different words: whoever takes it has first seen every bit below its own
// position, so a lower neighbour that could still read too few of them has made
// its own edge dead and does not ask, and for a higher one the taker's bit is
// never set.
#include <cstdint>

#include "amg_device.hpp"
#include "amg_internal.hpp"

namespace amg {

namespace {
constexpr int BS = 256;
inline int blocks_for(int64_t work, int bs = BS, int cap = 1 << 30) {
    int64_t b = (work + bs - 1) / bs;
    if (b < 1) b = 1;
    return (int)(b < cap ? b : cap);
}

__device__ __forceinline__ int find_col(const int* __restrict__ ci, int lo, int hi, int c) {
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        const int x = ci[mid];
        if (x == c) return mid;
        if (x < c) lo = mid + 1;
        else hi = mid;
    }
    return -1;
}

constexpr int INIT_GRP = 4;  // row entries whose loads k_hem_init issues together

// Position of column c in ci[lo, hi) (ascending), or -1: rows of up to 8
// entries in one load step, longer ones by bisection.
__device__ __forceinline__ int find_col_short(const int* __restrict__ ci, int lo, int hi, int c) {
    if (hi - lo > 8) return find_col(ci, lo, hi, c);
    int x[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) x[t] = lo + t < hi ? ci[lo + t] : -1;
    int p = -1;
#pragma unroll
    for (int t = 7; t >= 0; --t)
        if (x[t] == c) p = lo + t;
    return p;
}

// Up to 31 lower edges fit a word.  The lower edges of a vertex with more
// ("wide") have their bits in words of the extension array; its own word then
// holds the two summary states only.
constexpr int kWordEdges = 31;
// whether vertex j, with row ci[b, e), is wide
__device__ __forceinline__ bool wide_row(const int* __restrict__ ci, int b, int e, int j) {
    return e - b > kWordEdges && ci[b + kWordEdges] < j;
}
constexpr unsigned kTaken = 0x80000000u;
constexpr unsigned kAllDead = 0x7fffffffu;
constexpr int kWideFlag = 1 << 31;  // deg[].x: offset into the extension array
constexpr int kZeroFlag = 1 << 30;  // deg[].y: the row stores zeros above the diagonal
// Record entry: distance to the neighbour << 5 | position of the vertex among
// the neighbour's lower edges.  0 ends the list; kRowEnt says that the rest
// of the list has to be read from the row (a wide neighbour, or one too far).
constexpr int kMaxDelta = 1 << 26;
constexpr int kRowEnt = 31;
// Where a vertex is in the row of a higher edge-neighbour, per entry of its own
// row: kHas | position, and kWideEnt if the neighbour is wide.  0: no such edge.
constexpr int kWideEnt = 1 << 31, kHas = 1 << 30;
__device__ __forceinline__ unsigned low_bits(int p) { return (1u << p) - 1u; }
}  // namespace

// Per vertex y of a pass: its record (the first 4, 16 or 32 higher edge-neighbours by
// |a_yj| descending, column ascending on ties), deg = (number of lower stored
// entries or extension offset | kWideFlag, number of higher edge-neighbours |
// kZeroFlag), its word for the other tiles (0) and mate (-1).
// counters: cnt[1] words of the extension array used, cnt[5] sum over rows of
// (#upper - #lower) entries; err: an upper entry whose mirror image is not
// stored.  Together these are zero exactly for a symmetric pattern.
constexpr int kInitList = 4;
__global__ __launch_bounds__(BS) void k_hem_init(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                                                 const double* __restrict__ v, int* __restrict__ rec,
                                                 int2* __restrict__ deg, unsigned* __restrict__ gw,
                                                 unsigned* __restrict__ xw, int* __restrict__ mate, int* cnt,
                                                 int* err) {
    const int y = blockIdx.x * BS + threadIdx.x;
    int nlow = 0, nup = 0;
    if (y < n) {
        mate[y] = -1;
        gw[y] = 0u;
        int nh = 0, bad = 0, zero = 0;
        int ent[kInitList];
        double wt[kInitList];
#pragma unroll
        for (int t = 0; t < kInitList; ++t) {
            ent[t] = 0;
            wt[t] = 0.0;
        }
        // Entries in groups of INIT_GRP: the loads of a group (columns, values,
        // the rows of the higher neighbours) are issued together, then the
        // entries are taken in order.
        const int e0 = rp[y], e1 = rp[y + 1];
        for (int k0 = e0; k0 < e1; k0 += INIT_GRP) {
            int us[INIT_GRP], pos[INIT_GRP];
            double own[INIT_GRP];
            bool wide[INIT_GRP];
#pragma unroll
            for (int t = 0; t < INIT_GRP; ++t) {
                us[t] = k0 + t < e1 ? ci[k0 + t] : y;
                own[t] = k0 + t < e1 ? v[k0 + t] : 0.0;
            }
#pragma unroll
            for (int t = 0; t < INIT_GRP; ++t) {
                pos[t] = -1;
                wide[t] = false;
                if (us[t] > y) {
                    const int b = rp[us[t]], e = rp[us[t] + 1];
                    const int at = find_col_short(ci, b, e, y);
                    pos[t] = at < 0 ? -1 : at - b;
                    wide[t] = wide_row(ci, b, e, us[t]);
                }
            }
#pragma unroll
            for (int q = 0; q < INIT_GRP; ++q) {
                if (k0 + q >= e1) break;
                const int u = us[q];
                nlow += u < y;
                if (u <= y) continue;
                ++nup;
                if (pos[q] < 0) {
                    bad = 1;
                    continue;
                }
                const double w = fabs(own[q]);
                if (w == 0.0) {
                    zero = 1;
                    continue;
                }
                ++nh;
                const int delta = u - y;
                const int code = wide[q] || delta >= kMaxDelta ? kRowEnt : (delta << 5) | pos[q];
                int at = 0;  // by |a| descending; columns arrive ascending
#pragma unroll
                for (int t = 0; t < kInitList; ++t)
                    if (t < nh - 1 && wt[t] >= w) at = t + 1;
#pragma unroll
                for (int t = kInitList - 1; t > 0; --t)
                    if (t > at) {  // a full list drops its last entry
                        wt[t] = wt[t - 1];
                        ent[t] = ent[t - 1];
                    }
#pragma unroll
                for (int t = 0; t < kInitList; ++t)
                    if (t == at) {
                        wt[t] = w;
                        ent[t] = code;
                    }
            }
        }
        int4* out = reinterpret_cast<int4*>(rec) + (size_t)y * (kInitList / 4);
#pragma unroll
        for (int t = 0; t < kInitList; t += 4) out[t / 4] = make_int4(ent[t], ent[t + 1], ent[t + 2], ent[t + 3]);
        int low = nlow;
        if (nlow > kWordEdges) {  // extension: the number of lower entries, then their bits
            const int words = (nlow + 31) / 32;
            const int at = atomicAdd(&cnt[1], 1 + words);
            xw[at] = (unsigned)nlow;
            for (int k = 0; k < words; ++k) xw[at + 1 + k] = nlow - 32 * k >= 32 ? 0u : ~low_bits(nlow - 32 * k);
            low = at | kWideFlag;
        }
        deg[y] = make_int2(low, nh | (zero ? kZeroFlag : 0));
        if (bad) atomicOr(err, ERR_NONSYM);
    }
    // The pattern check, summed over the block and added only when nonzero:
    // adds to one word from every block serialise across the XCDs.  With one
    // add per wave, the first pass of a 128^3 grid (where every wave holds a
    // row at the end of a grid line) took 1.83 ms instead of 1.56 ms; a
    // block's boundary rows mostly cancel.
    __shared__ int s_diff[BS / kWave];
    int diff = nup - nlow;
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) diff += __shfl_xor(diff, o);
    if (threadIdx.x % kWave == 0) s_diff[threadIdx.x / kWave] = diff;
    __syncthreads();
    if (threadIdx.x == 0) {
        int d = 0;
#pragma unroll
        for (int k = 0; k < BS / kWave; ++k) d += s_diff[k];
        if (d != 0) atomicAdd(&cnt[5], d);
    }
}

// The same with G lanes a row, an entry a lane or two; for all but the largest
// regular levels, where a thread a row above is faster.  An entry's place in
// the record is its rank among the row's, counted through LDS (weights compare
// as their bit patterns: a strict order, with the column, whatever they are).
// Rows of more than 2 G entries are ranked by taking the largest R times.
// A row whose list the record does not hold leaves where its mirror images are in
// ent, an int per entry, so that the matching need not look for them each time.
// Every entry's mirror image is looked for, the lower ones' by lanes that would
// wait, so no sum over the rows is needed: with one add a block to a single
// word a pass of 65,536 rows took 53 us instead of 13.
//
// Bound by the chain of loads down to the neighbours' rows.  With a thread a
// row, inserting into a list of 16 or 32 in registers, any small level of 12-20
// entries a row took 45-80 us; this takes 6-12, and 22 at 55,000 rows (57), 28 at
// 110,000 (39).
namespace {
struct InitRow {  // what a row's lanes find together
    int nlow, nh;
    bool zero, bad;
};

// y in the row of its neighbour u: code of y's record entry for u, and where it
// is (kHas | position, and kWideEnt if u is wide; 0: u's row has no y)
struct InitEdge {
    int code, at;
};
__device__ __forceinline__ InitEdge init_edge(const int* __restrict__ rp, const int* __restrict__ ci, int y, int u) {
    const int b = rp[u], e = rp[u + 1];
    const int pos = find_col_short(ci, b, e, y) - b;
    const int delta = u - y;
    const bool wide = wide_row(ci, b, e, u);
    return InitEdge{wide || delta >= kMaxDelta ? kRowEnt : (delta << 5) | pos,
                    pos >= 0 ? kHas | pos | (wide ? kWideEnt : 0) : 0};
}

__device__ __forceinline__ unsigned long long weight_bits(double a) { return (unsigned long long)__double_as_longlong(fabs(a)); }

template <int R, int G, int E>
__device__ __forceinline__ InitRow init_row(int y, int e0, int L, const int* __restrict__ rp,
                                            const int* __restrict__ ci, const double* __restrict__ v,
                                            unsigned long long* key, int* __restrict__ out, int* __restrict__ ent) {
    const int lane = threadIdx.x & (G - 1), base = threadIdx.x & (kWave - 1) & ~(G - 1);
    const unsigned group = unsigned((1ull << G) - 1);
    int u[E];
    InitEdge in[E];
    double a[E];
    unsigned long long w[E];
#pragma unroll
    for (int t = 0; t < E; ++t) {
        const int k = lane + G * t;
        u[t] = k < L ? ci[e0 + k] : y;
        a[t] = k < L ? v[e0 + k] : 0.0;
    }
    InitRow r{0, 0, false, false};
    bool other = false;  // an entry that a record cannot hold
#pragma unroll
    for (int t = 0; t < E; ++t) {
        in[t] = InitEdge{0, 0};
        const bool off = u[t] != y;
        if (off) in[t] = init_edge(rp, ci, y, u[t]);
        const bool ok = in[t].at != 0;
        const bool up = ok && u[t] > y;
        w[t] = up ? weight_bits(a[t]) : 0;
        key[lane + G * t] = w[t];
        r.nlow += __popc(unsigned(__ballot(u[t] < y) >> base) & group);
        r.nh += __popc(unsigned(__ballot(w[t] != 0) >> base) & group);
        r.zero |= (unsigned(__ballot(up && w[t] == 0) >> base) & group) != 0;
        r.bad |= (unsigned(__ballot(off && !ok) >> base) & group) != 0;
        other |= (unsigned(__ballot(w[t] != 0 && in[t].code == kRowEnt) >> base) & group) != 0;
    }
    if (ent && (r.nh > R || other)) {  // a row that the record does not hold
#pragma unroll
        for (int t = 0; t < E; ++t)
            if (lane + G * t < L) ent[e0 + lane + G * t] = w[t] != 0 ? in[t].at : 0;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    int rank[E] = {};
    for (int j = 0; j < L; j += 2) {  // a place past the row holds 0
        const ulonglong2 q = *reinterpret_cast<const ulonglong2*>(key + j);
#pragma unroll
        for (int t = 0; t < E; ++t) {
            const int k = lane + G * t;
            rank[t] += (q.x > w[t] || (q.x == w[t] && j < k)) + (q.y > w[t] || (q.y == w[t] && j + 1 < k));
        }
    }
#pragma unroll
    for (int t = 0; t < E; ++t)
        if (w[t] != 0 && rank[t] < R) out[rank[t]] = in[t].code;
    for (int q = lane; q < R; q += G)
        if (q >= r.nh) out[q] = 0;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    return r;
}

template <int R, int G>
__device__ __forceinline__ InitRow init_long_row(int y, int e0, int L, const int* __restrict__ rp,
                                                 const int* __restrict__ ci, const double* __restrict__ v,
                                                 int* __restrict__ out, int* __restrict__ ent) {
    const int lane = threadIdx.x & (G - 1);
    InitRow r{0, 0, false, false};
    for (int k = lane; k < L; k += G) {
        const int u = ci[e0 + k];
        r.nlow += u < y;
        int at = 0;
        if (u != y) {
            at = init_edge(rp, ci, y, u).at;
            if (at == 0) r.bad = true;
            if (u < y) at = 0;
            else if (weight_bits(v[e0 + k]) == 0) {
                r.zero |= at != 0;
                at = 0;
            }
        }
        r.nh += at != 0;
        if (ent) ent[e0 + k] = at;
    }
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) {
        r.nlow += __shfl_xor(r.nlow, o, G);
        r.nh += __shfl_xor(r.nh, o, G);
        r.zero |= __shfl_xor((int)r.zero, o, G) != 0;
        r.bad |= __shfl_xor((int)r.bad, o, G) != 0;
    }
    unsigned long long pw = ~0ull;
    int pk = -1;  // the entry taken last
    for (int q = 0; q < R; ++q) {
        unsigned long long bw = 0;
        int bk = L;
        for (int k = lane; k < L; k += G) {
            if (ci[e0 + k] <= y) continue;
            const unsigned long long w = weight_bits(v[e0 + k]);
            if ((w < pw || (w == pw && k > pk)) && w > bw) {
                bw = w;
                bk = k;
            }
        }
#pragma unroll
        for (int o = G / 2; o > 0; o >>= 1) {
            const unsigned long long ow = __shfl_xor(bw, o, G);
            const int ok = __shfl_xor(bk, o, G);
            if (ow > bw || (ow == bw && ok < bk)) {
                bw = ow;
                bk = ok;
            }
        }
        int code = 0;
        if (bw != 0) code = init_edge(rp, ci, y, ci[e0 + bk]).code;
        if (lane == 0) out[q] = code;
        pw = bw;
        pk = bk;
    }
    return r;
}

constexpr int kInitBlocks = 4096;   // two rounds of the chip
constexpr int kInitThread = 32768;  // levels of few entries a row above this take a thread a row (7 us here, 13 against 7 at 65,536)
}  // namespace

template <int R, int G>
__global__ __launch_bounds__(BS) void k_hem_init_group(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                                                       const double* __restrict__ v, int* __restrict__ rec,
                                                       int2* __restrict__ deg, unsigned* __restrict__ gw,
                                                       unsigned* __restrict__ xw, int* __restrict__ mate, int* cnt,
                                                       int* err, int* __restrict__ ent) {
    __shared__ __align__(16) unsigned long long skey[2 * BS];
    const int g = threadIdx.x / G, lane = threadIdx.x & (G - 1);
    unsigned long long* key = skey + g * 2 * G;
    for (int y = blockIdx.x * (BS / G) + g; y < n; y += gridDim.x * (BS / G)) {
        const int e0 = rp[y], L = rp[y + 1] - e0;
        int* out = rec + (size_t)y * R;
        const InitRow r = L <= G       ? init_row<R, G, 1>(y, e0, L, rp, ci, v, key, out, ent)
                          : L <= 2 * G ? init_row<R, G, 2>(y, e0, L, rp, ci, v, key, out, ent)
                                       : init_long_row<R, G>(y, e0, L, rp, ci, v, out, ent);
        if (lane == 0) {
            mate[y] = -1;
            gw[y] = 0u;
            int low = r.nlow;
            if (r.nlow > kWordEdges) {  // extension: the number of lower entries, then their bits
                const int words = (r.nlow + 31) / 32;
                const int at = atomicAdd(&cnt[1], 1 + words);
                xw[at] = (unsigned)r.nlow;
                for (int k = 0; k < words; ++k)
                    xw[at + 1 + k] = r.nlow - 32 * k >= 32 ? 0u : ~low_bits(r.nlow - 32 * k);
                low = at | kWideFlag;
            }
            deg[y] = make_int2(low, r.nh | (r.zero ? kZeroFlag : 0));
            if (r.bad) atomicOr(err, ERR_NONSYM);
        }
    }
}

namespace {
struct HemState {
    int n;
    const int* __restrict__ rp;
    const int* __restrict__ ci;
    const double* __restrict__ v;
    const int* __restrict__ rec;
    const int2* __restrict__ deg;
    const int* __restrict__ ent;  // per entry of rows that their records do not hold: its mirror image; or null
    unsigned* gw;  // words set by other tiles
    unsigned* xw;  // extension words of wide vertices
    int* mate;
};

__device__ __forceinline__ unsigned load_dev(const unsigned* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void or_dev(unsigned* p, unsigned bits) {
    (void)__hip_atomic_fetch_or(p, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// All memory operations of the wave have completed.  Ends each rare path that
// loads from global memory: a load that the compiler takes to be outstanding
// at the head of the sweep makes every sweep wait for the wave's stores.
__device__ __forceinline__ void settle() { __builtin_amdgcn_s_waitcnt(0x0f70); }  // vmcnt(0)

// Whether the pass was given up (the same for the whole wave).
__device__ __forceinline__ bool given_up(const int* cnt) {
    const int g = __hip_atomic_load(&cnt[7], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return __builtin_amdgcn_readfirstlane(g) != 0;
}

// LDS words that other waves of the workgroup read or write meanwhile
template <class I>
__device__ __forceinline__ I lds_load(const I* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
template <class I>
__device__ __forceinline__ void lds_store(I* p, I x) {
    __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
template <class I>
__device__ __forceinline__ void lds_or(I* p, I bits) {
    (void)__hip_atomic_fetch_or(p, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

enum { kUnknown = 0, kAvail = 1, kGone = 2 };

// What is known of a vertex's choices in higher tiles: low half, a bit per record
// entry that its state is known; high half, that it is available.  One word, so
// that no read has the first without the second (read apart, a known entry that
// looks unavailable would be passed by).  The low half is also watched as a word.
using Known = unsigned long long __attribute__((may_alias));

// The tile of a workgroup: vertices off .. off + m - 1, their words in LDS.
// The bits of lower edges from other tiles arrive in gw (set there by those
// tiles) and are merged into the LDS word by a polling wave; a
// lower tile reads a vertex's state from gw alone, since all lower edges below
// its own come from its own tile or lower ones.
struct Tile {
    int off, m;
    unsigned* w;
    __device__ __forceinline__ bool mine(int i) const { return (unsigned)(i - off) < (unsigned)m; }
    __device__ __forceinline__ unsigned load(int i) const {
        return lds_load(&w[i]);
    }
    __device__ __forceinline__ void set(int i, unsigned bits) const {
        lds_or(&w[i], bits);
    }
    __device__ __forceinline__ unsigned word(const HemState& S, int j) const {
        return mine(j) ? load(j - off) : load_dev(&S.gw[j]);
    }
    __device__ __forceinline__ void set_word(const HemState& S, int j, unsigned bits) const {
        if (mine(j)) set(j - off, bits);
        else or_dev(&S.gw[j], bits);
    }
    // lower edge `pos` of j is dead
    __device__ __forceinline__ void dead(const HemState& S, int j, int pos, bool wide) const {
        if (!wide) set_word(S, j, 1u << pos);
        else or_dev(&S.xw[(S.deg[j].x & ~kWideFlag) + 1 + pos / 32], 1u << (pos % 32));
    }
    // lower edge `pos` of j, with extension words xo, is taken
    __device__ __forceinline__ void taken(const HemState& S, int j, int pos, int xo) const {
        if (xo < 0) {
            set_word(S, j, ~(1u << pos));
            return;
        }
        set_word(S, j, kTaken);
        const int words = ((int)S.xw[xo - 1] + 31) / 32;
        for (int k = 0; k < words; ++k) or_dev(&S.xw[xo + k], k == pos / 32 ? ~(1u << (pos % 32)) : ~0u);
    }
    // a wide vertex's extension words (-1: the vertex is not wide)
    __device__ __forceinline__ int ext(const HemState& S, int j, bool wide) const {
        return wide ? (S.deg[j].x & ~kWideFlag) + 1 : -1;
    }
    // a vertex for its lower edge `pos`, from its word wj and extension words xo
    __device__ __forceinline__ int state(const HemState& S, int pos, int xo, unsigned wj) const {
        bool full;
        if (xo < 0) {
            full = (~wj & low_bits(pos)) == 0u;
        } else {
            full = true;
            for (int k0 = 0; 32 * k0 < pos && full; k0 += 4) {  // four loads in flight
                unsigned x[4];
                const int last = (pos - 1) / 32;
#pragma unroll
                for (int k = 0; k < 4; ++k) x[k] = load_dev(&S.xw[xo + min(k0 + k, last)]);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int need = pos - 32 * min(k0 + k, last);
                    full &= (~x[k] & (need >= 32 ? ~0u : low_bits(need))) == 0u;
                }
            }
            settle();
        }
        return full ? kAvail : (wj & kTaken) ? kGone : kUnknown;
    }
};

// Entry e of u's row, as kHas | .. above; j: its column.
__device__ __forceinline__ int row_edge(const HemState& S, int u, int e, int j) {
    if (S.ent) return S.ent[e];
    if (j <= u || S.v[e] == 0.0) return 0;
    const int b = S.rp[j], e1 = S.rp[j + 1];
    return kHas | (find_col(S.ci, b, e1, u) - b) | (wide_row(S.ci, b, e1, j) ? kWideEnt : 0);
}
__device__ __forceinline__ int edge_pos(int at) { return at & (kHas - 1); }

// A vertex's choice from its row: the neighbour (-1: none), its position and
// extension words, and its state.
struct RowChoice {
    int j, pos, xo, st;
};

// By a whole wave, on one vertex u with row entries b .. e1 - 1: its heaviest
// higher edge-neighbour not known to be unavailable (lowest column on ties).
__device__ __forceinline__ RowChoice wave_choice(const HemState& S, const Tile& T, int u, int b, int e1) {
    const int lane = threadIdx.x % kWave;
    unsigned long long bw = 0;
    int bj = INT_MAX, bp = 0, bs = kUnknown, bx = -1;
    for (int e = b + lane; e < e1; e += kWave) {
        const int j = S.ci[e], at = row_edge(S, u, e, j);
        // non-negative doubles order as their bits do; every weight is nonzero
        const unsigned long long w = weight_bits(S.v[e]);
        if (at == 0) continue;
        const int xo = T.ext(S, j, at < 0);
        const int s = T.state(S, edge_pos(at), xo, T.word(S, j));
        if (s != kGone && (w > bw || (w == bw && j < bj))) {
            bw = w;
            bj = j;
            bp = edge_pos(at);
            bs = s;
            bx = xo;
        }
    }
    unsigned long long mw = bw;
    int mj = bj;
    for (int o = kWave / 2; o > 0; o >>= 1) {
        const unsigned long long ow = __shfl_xor(mw, o);
        const int oj = __shfl_xor(mj, o);
        if (ow > mw || (ow == mw && oj < mj)) {
            mw = ow;
            mj = oj;
        }
    }
    if (mj == INT_MAX) return RowChoice{-1, 0, -1, kGone};
    const int src = __ffsll((long long)__ballot(bj == mj)) - 1;  // each column is held by one lane
    return RowChoice{mj, __builtin_amdgcn_readlane(bp, src), __builtin_amdgcn_readlane(bx, src),
                     __builtin_amdgcn_readlane(bs, src)};
}

// By a whole wave: every higher edge of u (row entries b .. e1 - 1) but the one
// to `keep` is dead.
__device__ __forceinline__ void wave_dead(const HemState& S, const Tile& T, int u, int b, int e1, int keep) {
    constexpr int B = 4;  // entries of a lane in flight together
    for (int e0 = b + (int)(threadIdx.x % kWave); e0 < e1; e0 += B * kWave) {
        int j[B], at[B];
#pragma unroll
        for (int k = 0; k < B; ++k) {
            const int e = e0 + k * kWave;
            j[k] = e < e1 ? S.ci[e] : keep;
            at[k] = e < e1 ? row_edge(S, u, e, j[k]) : 0;
        }
#pragma unroll
        for (int k = 0; k < B; ++k)
            if (at[k] != 0 && j[k] != keep) T.dead(S, j[k], edge_pos(at[k]), at[k] < 0);
    }
}

// State of a vertex: its current choice's record entry (16 bits) and these flags
enum : unsigned {
    vConf = 1u << 16,  // the current choice is available: later edges are dead
    vRow = 1u << 17,   // past the record: choices come from the row
    vWide = 1u << 18,  // the vertex itself is wide
    vMore = 1u << 19,  // the record does not hold the whole list
    vRare = 1u << 20,  // waits for words that only the wave itself polls
    vDone = 1u << 21,
};
constexpr unsigned kNever = ~0u;
constexpr int kNoRest = -2;  // no edges of the row are left to mark

// Bits of p over the group of G lanes that this lane is in.
template <int G>
__device__ __forceinline__ unsigned group_mask(bool p) {
    const unsigned long long b = __ballot(p) >> ((threadIdx.x % kWave) & ~(G - 1));
    return (unsigned)b & (G == 32 ? ~0u : (1u << (G % 32)) - 1u);
}

// The polling waves of a tile; they end when every other wave has.  The first
// merges the bits that lower tiles set in this tile's words into LDS.
template <int TM>
__device__ __forceinline__ void poll_words(const HemState& S, const Tile& T, const unsigned* s_m, const int* s_left) {
    constexpr int B = TM / kWave;  // vertices of a lane, their loads in flight together
    const int lane = threadIdx.x % kWave;
    unsigned need[B];
#pragma unroll
    for (int i = 0; i < B; ++i) need[i] = lane + i * kWave < T.m ? s_m[lane + i * kWave] : 0u;
    __builtin_amdgcn_s_setprio(3);
    while (lds_load(s_left) > 0) {
        unsigned g[B], any = 0u;
#pragma unroll
        for (int i = 0; i < B; ++i) {
            g[i] = need[i] ? load_dev(&S.gw[T.off + lane + i * kWave]) : 0u;
            any |= need[i];
        }
        if (__ballot(any != 0u) == 0) break;
#pragma unroll
        for (int i = 0; i < B; ++i) {
            if (g[i] & (need[i] | kTaken)) T.set(lane + i * kWave, g[i]);
            need[i] = g[i] & kTaken ? 0u : need[i] & ~g[i];
        }
    }
}

// The second looks up the choices in higher tiles that are waited for: those
// of vertices that are free to take them each time, the others, which only
// let later edges be marked earlier, every eighth time.
template <int TM>
__device__ __forceinline__ void poll_choices(const HemState& S, const Tile& T, Known* s_k, const int* s_r,
                                             const int* s_e, const int* s_left) {
    constexpr int B = TM / kWave < 8 ? TM / kWave : 8;
    const int lane = threadIdx.x % kWave;
    __builtin_amdgcn_s_setprio(3);
    for (int it = 0; lds_load(s_left) > 0; ++it) {
        bool idle = true;
        for (int l0 = lane; l0 - lane < T.m; l0 += B * kWave) {
            unsigned t[B];
            int r[B], q[B];
            bool any = false;
#pragma unroll
            for (int i = 0; i < B; ++i) {
                const int l = l0 + i * kWave;
                r[i] = 0;
                if (l < T.m) {
                    r[i] = lds_load(&s_r[l]);
                    if (r[i] > 0 && ((lds_load(&s_k[l]) >> (r[i] - 1)) & 1u)) r[i] = 0;
                    if ((it & 7) != 0 && T.load(l) != kAllDead) r[i] = 0;
                    q[i] = r[i] > 0 ? s_e[(r[i] - 1) * (TM + 1) + l] : 0;
                }
                any |= r[i] > 0;
            }
            if (__ballot(any) == 0) continue;
            idle = false;
#pragma unroll
            for (int i = 0; i < B; ++i)
                t[i] = r[i] > 0 ? load_dev(&S.gw[T.off + l0 + i * kWave + (q[i] >> 5)]) : 0u;
#pragma unroll
            for (int i = 0; i < B; ++i) {
                const int l = l0 + i * kWave;
                if (r[i] > 0) {
                    const bool full = (~t[i] & low_bits(q[i] & 31)) == 0u;
                    const Known bit = 1ull << (r[i] - 1);
                    if (full) lds_or(&s_k[l], bit | bit << 32);
                    else if (t[i] & kTaken) lds_or(&s_k[l], bit);
                }
            }
        }
        if (idle) __builtin_amdgcn_s_sleep(4);
    }
}

}  // namespace

// One workgroup per tile of `rows` vertices, one per thread of all waves but
// the last two, all tiles in one launch.  Tiles are handed out in ascending
// order as workgroups start, so every tile below a running one is running or
// done, and waiting on lower tiles ends.
//
// What bounds it: a pass is a chain of dependent decisions (about 300 of them
// on a 128^3 grid, 700 on smooth coefficients at 160^3), so its time is their
// number times the latency of one; neither memory nor arithmetic is near its
// limit.  A step inside a tile takes about 1 us, one to another tile 3 to 4 us
// (an atomic to memory, a poll, and the step there).  Hence:
//  * Waves run on their own, without barriers.  Each vertex watches two words
//    in LDS, its own and its current choice's, each with a mask: it is looked
//    at once a word has all bits of its mask, or the top bit.  A sweep over
//    them is two LDS reads and a few compares.
//  * The vertices found are taken a group of lanes each, a lane per record
//    entry (two with 32): the states of all choices, and the marking of all
//    edges, take one step each.  One lane per vertex took 12000 clocks a sweep
//    (the entries one after another), a whole wave per vertex 1700 a vertex; a
//    group step takes about 2000 for up to 4 vertices, or 16 with short rows.
//  * No wave that matches touches global memory but to store.  The last two
//    poll what other tiles set: bits of this tile's words are merged into LDS,
//    and for each choice in a higher tile that is waited for, s_k tells, per
//    record entry, that it is known and whether it is available.  Facts about an
//    entry stay true, so nothing is taken back when a vertex moves on.
//
// Against rounds of ready vertices between barriers (the same matching):
// the passes of a setup at 160^3 with smooth coefficients took 85 ms and take
// 15 ms, those at 128^3 (constant coefficients) 6.8 ms and 3.9 ms.
//
// Past tmo wall-clock ticks a wave stops and sets cnt[7]; the other waves look at
// it when they look at the clock, workgroups before they take a tile, so a pass
// given up has ended within about one limit whatever its number of tiles.  The
// host repeats it with a longer limit (every fact found is found again).
template <int R, int NT>
__global__ __launch_bounds__(NT) void k_hem_tile(HemState S, int rows, int* cnt, const int* err, long long tmo) {
    constexpr int TM = NT - 2 * kWave;  // vertices of a tile at most
    constexpr int G = R < 16 ? R : 16, E = R / G, NG = kWave / G;
    constexpr int ES = TM + 1;      // entry t of vertex l at s_e[t * ES + l]: no bank conflicts either way
    constexpr int KW = TM + 2;  // s_w from here on: s_k
    __shared__ __align__(8) unsigned s_w[KW + 2 * TM];  // words, one that is never looked at (and one more), s_k
    __shared__ unsigned s_m[TM];          // bits of lower edges from other tiles
    __shared__ int s_r[TM];               // 1 + the entry waited for in a higher tile
    __shared__ int s_e[R * ES];
    __shared__ int4 s_sel[TM / kWave * NG];
    __shared__ int s_tile, s_left, s_max;
    // a pattern that is not symmetric: some bits would never be set
    if (cnt[5] != 0 || (*err & ERR_NONSYM)) return;
    if (threadIdx.x == 0) {
        s_tile = given_up(cnt) ? -1 : atomicAdd(&cnt[0], 1);
        s_left = TM / kWave;
        s_max = 0;
        s_w[TM] = 0u;
    }
    __syncthreads();
    if (s_tile < 0) return;
    const int off = s_tile * rows;
    const int m = min(rows, S.n - off);
    const Tile T{off, m, s_w};
    const int lane = threadIdx.x % kWave, base = threadIdx.x - lane;
    const int l = threadIdx.x, u = off + l;
    Known* const s_k = reinterpret_cast<Known*>(s_w + KW);
    unsigned st = 0, mo = kNever, mt = kNever;
    int to = TM, ta = TM;
    bool zeros = false;
    int rb = 0, re = 0;  // the row
    if (l < m) {
        const int2 d = S.deg[u];
        const int b = S.rp[u];
        rb = b;
        re = S.rp[u + 1];
        const int c = d.y & ~kZeroFlag;
        zeros = (d.y & kZeroFlag) != 0;
        if (c > R) st |= vMore;
        unsigned w0 = 0u, xm = 0u;
        if (d.x & kWideFlag) {
            st |= vWide | vRare;
        } else {
            int nx = 0;  // lower edges from other tiles come first
            while (nx < d.x && S.ci[b + nx] < off) ++nx;
            xm = low_bits(nx);
            w0 = kAllDead & ~low_bits(d.x);
        }
        s_w[l] = w0;
        s_k[l] = 0u;
        s_m[l] = xm;
        s_r[l] = 0;
#pragma unroll
        for (int t = 0; t < R; t += 4) {
            const int4 q = reinterpret_cast<const int4*>(S.rec)[(size_t)u * (R / 4) + t / 4];
            if (q.x == kRowEnt || q.y == kRowEnt || q.z == kRowEnt || q.w == kRowEnt) st |= vMore;
            s_e[t * ES + l] = q.x;
            s_e[(t + 1) * ES + l] = q.y;
            s_e[(t + 2) * ES + l] = q.z;
            s_e[(t + 3) * ES + l] = q.w;
        }
        to = l;
        mt = 0u;  // looked at once to begin with
    }
    __syncthreads();
    if (zeros) {  // stored zeros are no edges: dead from the start
        for (int e = rb; e < re; ++e) {
            const int j = S.ci[e];
            if (j <= u || S.v[e] != 0.0) continue;
            const int b = S.rp[j], e1 = S.rp[j + 1];
            T.dead(S, j, find_col(S.ci, b, e1, u) - b, wide_row(S.ci, b, e1, j));
        }
    }
    if (base >= TM) {
        if (gridDim.x > 1 && base == TM) poll_words<TM>(S, T, s_m, &s_left);
        else if (gridDim.x > 1) poll_choices<TM>(S, T, s_k, s_r, s_e, &s_left);
        return;
    }
    // the edge of record entry q of LDS vertex b is dead
    auto mark = [&](int b, int q) {
        const int jl = b + (q >> 5);
        if (jl < m) T.set(jl, 1u << (q & 31));
        else or_dev(&S.gw[off + jl], 1u << (q & 31));
    };
    int xa = 0, xe = 0;  // a wide vertex's extension words, those known to be full left out
    if (st & vWide) {
        xa = (S.deg[u].x & ~kWideFlag) + 1;
        xe = xa + ((int)S.xw[xa - 1] + 31) / 32;
    }
    int cj = -1, cp = 0, cx = -1;  // the choice from the row: vertex, position, extension words
    int4* const sel = s_sel + base / kWave * NG;
    const long long t_start = wall_clock64();
    int sweeps = 0;
    bool late = false;
    for (;;) {
        const unsigned own = T.load(to), tgt = T.load(ta);
        const bool fire = (~own & mo) == 0u || (~tgt & mt) == 0u || (int)own < 0 || (int)tgt < 0;
        unsigned long long todo = __ballot(fire);
        if ((++sweeps & 1023) == 0 && (wall_clock64() - t_start > tmo || given_up(cnt))) {
            late = true;
            break;
        }
        if (todo == 0) {
            if (__ballot(to != TM) == 0) break;
            if (__ballot((st & vRare) != 0) != 0) {
                // wide vertices and choices from the row: their words in global memory
                if ((st & vWide) && to != TM) {
                    // the words from the first that was not full, four at a time
                    const unsigned g0 = load_dev(&S.gw[u]);
                    unsigned x[4];
                    bool on;
                    do {
#pragma unroll
                        for (int i = 0; i < 4; ++i) x[i] = load_dev(&S.xw[min(xa + i, xe - 1)]);
                        on = (x[0] & x[1] & x[2] & x[3]) == ~0u;
                        if (on) xa = min(xa + 4, xe);
                    } while (on && xa < xe);
                    const unsigned g = g0 | (xa == xe ? kAllDead : 0u);
                    if (g != 0u) T.set(l, g);
                }
                if ((st & vRow) && !(st & vConf) && to != TM && cj >= 0 && T.state(S, cp, cx, T.word(S, cj)) != kUnknown)
                    mt = 0u;
                settle();
            }
            __builtin_amdgcn_s_sleep(2);
            continue;
        }
        __builtin_amdgcn_s_setprio(2);  // before the waves that only look
        if (__ballot(fire && (st & vRow)) != 0) {
            // choices from the row: one vertex at a time, by the whole wave
            unsigned long long row = __ballot(fire && (st & vRow));
            todo &= ~row;
            while (row != 0) {
                const int src = __ffsll((long long)row) - 1;
                row &= row - 1;
                const unsigned ow = __builtin_amdgcn_readlane(own, src);
                unsigned f = __builtin_amdgcn_readlane(st, src);
                RowChoice c{__builtin_amdgcn_readlane(cj, src), __builtin_amdgcn_readlane(cp, src),
                            __builtin_amdgcn_readlane(cx, src), kGone};
                const int b = __builtin_amdgcn_readlane(rb, src), e1 = __builtin_amdgcn_readlane(re, src);
                const int v = off + base + src;
                bool done = false;
                if (ow & kTaken) {
                    wave_dead(S, T, v, b, e1, -1);
                    done = true;
                } else {
                    if (!(f & vConf)) {
                        // one lane's reading: words change meanwhile, and lanes that
                        // read differently would take different branches
                        if (c.j >= 0)
                            c.st = __builtin_amdgcn_readfirstlane(T.state(S, c.pos, c.xo, T.word(S, c.j)));
                        if (c.st == kGone) c = wave_choice(S, T, v, b, e1);
                        if (c.j < 0) {
                            f |= vConf;  // no neighbour left
                        } else if (c.st == kAvail) {
                            f |= vConf;
                            wave_dead(S, T, v, b, e1, c.j);
                        }
                    }
                    if (ow == kAllDead && (f & vConf)) {
                        if (c.j >= 0 && lane == 0) {
                            S.mate[v] = c.j;
                            S.mate[c.j] = v;
                            T.taken(S, c.j, c.pos, c.xo);
                        }
                        if (c.j >= 0 && c.xo < 0 && c.j < off + m) {
                            const int q = lane < R ? s_e[lane * ES + (c.j - off)] : 0;
                            if (q > kRowEnt) mark(c.j - off, q);
                        }
                        done = true;
                    }
                }
                if (lane == src) {
                    st = f | vRare;
                    cj = c.j;
                    cp = c.pos;
                    cx = c.xo;
                    ta = TM;
                    mt = kNever;
                    mo = f & vConf ? kAllDead : kNever;
                    if (done) {
                        to = TM;
                        mo = kNever;
                    }
                }
            }
            settle();
        }
        // the others, NG at a time: a group of G lanes each, E record entries a lane
        const int rank = __builtin_amdgcn_mbcnt_hi((unsigned)(todo >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)todo, 0u));
        const bool mine = (todo >> lane) & 1u;
        const int total = __popcll(todo);
        int more = kNoRest;
        for (int r0 = 0; r0 < total; r0 += NG) {
            const bool turn = mine && rank >= r0 && rank < r0 + NG;
            if (turn) sel[rank - r0] = make_int4(lane, (int)own, (int)st, 0);
            __builtin_amdgcn_wave_barrier();
            const int4 in = sel[lane / G];
            const bool live = r0 + lane / G < total;
            const int lv = base + (live ? in.x : 0), t = lane % G;
            const unsigned ow = live ? (unsigned)in.y : 0u, f = (unsigned)in.z;
            const int k0 = (int)(f & 0xffffu);
            const bool tk = (ow & kTaken) != 0u, conf = (f & vConf) != 0u;
            const Known known = lds_load(&s_k[lv]);
            const unsigned kn = (unsigned)known, av = (unsigned)(known >> 32), xm = s_m[lv];
            int q[E], jl[E];
            unsigned cm = 0u, fm = 0u, rm = 0u;  // entries: candidates, available ones, ones that the row holds
#pragma unroll
            for (int i = 0; i < E; ++i) {
                q[i] = live ? s_e[(t + i * G) * ES + lv] : 0;
                jl[i] = lv + (q[i] >> 5);
            }
#pragma unroll
            for (int i = 0; i < E; ++i) {
                const int e = t + i * G;
                const unsigned w = T.load(jl[i] < m ? jl[i] : TM);
                const bool full = (~w & low_bits(q[i] & 31)) == 0u || (av >> e) & 1u;
                const bool gone = !full && (jl[i] < m ? (int)w < 0 : ((kn >> e) & 1u) != 0u);
                cm |= group_mask<G>(q[i] != 0 && (conf ? e == k0 : e >= k0 && (q[i] == kRowEnt || !gone))) << (i * G);
                fm |= group_mask<G>(full) << (i * G);
                rm |= group_mask<G>(q[i] == kRowEnt) << (i * G);
            }
            const int k = cm != 0u ? __ffs(cm) - 1 : R;
            const unsigned bk = cm & (0u - cm);  // its bit, or none
            const bool row = !tk && !conf && ((rm & bk) != 0u || (cm == 0u && (f & vMore)));
            const bool nconf = !tk && !conf && !row && (cm == 0u || (fm & bk) != 0u);
            const bool all = tk && ((f & vWide) || ((xm >> ((__ffs(~ow) - 1) & 31)) & 1u));  // no taker of this tile did it
            const bool take = (conf || nconf) && !tk && ow == kAllDead;
            int kl = -1;  // the choice's LDS index, in the lane that holds its entry
#pragma unroll
            for (int i = 0; i < E; ++i) {
                const int e = t + i * G;
                if (q[i] > kRowEnt && (all || (nconf && e > k))) mark(lv, q[i]);
                if (e == k) kl = jl[i];
                if (e == k && take) {
                    S.mate[off + lv] = off + jl[i];
                    S.mate[off + jl[i]] = off + lv;
                    T.set_word(S, off + jl[i], ~(1u << (q[i] & 31)));
                }
            }
            if (__ballot(take) != 0) {  // the taken ones' edges are dead too: marked here, their ends see it one step earlier
                const int kt = __shfl(kl, (lane & ~(G - 1)) + (k & (G - 1)));
#pragma unroll
                for (int i = 0; i < E; ++i) {
                    const int q2 = take && cm != 0u && kt < m ? s_e[(t + i * G) * ES + kt] : 0;
                    if (q2 > kRowEnt) mark(kt, q2);
                }
            }
            if (live && t == (k & (G - 1))) {  // k = R: lane 0
                const bool done = tk || take;
                int nta = TM;
                unsigned nmt = row ? 0u : kNever;
                if (!done && !conf && !nconf && !row) {
                    nta = kl < m ? kl : KW + 2 * lv;
                    nmt = 1u << (k & 31);
#pragma unroll
                    for (int i = 0; i < E; ++i)
                        if (t + i * G == k && kl < m) nmt = low_bits(q[i] & 31);
                    if (kl >= m) lds_store(&s_r[lv], k + 1);
                }
                const unsigned nf = (f & ~0xffffu) | (unsigned)k | (nconf ? vConf : 0u) | (row ? vRow : 0u) | (done ? vDone : 0u);
                const int rest = !(f & vMore) ? kNoRest : tk ? -1 : nconf ? off + kl : kNoRest;
                sel[lane / G] = make_int4((int)nf, nta, (int)nmt, rest);
            }
            __builtin_amdgcn_wave_barrier();
            if (turn) {
                const int4 o = sel[rank - r0];
                st = (unsigned)o.x;
                ta = o.y;
                mt = (unsigned)o.z;
                more = o.w;
                mo = st & vDone ? kNever : st & vConf ? kAllDead : kNever;
                if (st & vDone) to = TM;
            }
        }
        if (__ballot(more != kNoRest) != 0) {
            unsigned long long rest = __ballot(more != kNoRest);
            while (rest != 0) {
                const int src = __ffsll((long long)rest) - 1;
                rest &= rest - 1;
                wave_dead(S, T, off + base + src, __builtin_amdgcn_readlane(rb, src),
                          __builtin_amdgcn_readlane(re, src), __builtin_amdgcn_readlane(more, src));
            }
            settle();
        }
        __builtin_amdgcn_s_setprio(0);
    }
    if (lane == 0) {
        if (late) atomicOr(&cnt[7], 1);
        atomicMax(&s_max, sweeps);
        if (atomicSub(&s_left, 1) == 1)
            atomicMax(&cnt[6], lds_load(&s_max));
    }
}

// ---------------------------------------------------------------------------
// Edge-based matching (Algorithm 3): the greedy matching over undirected
// edges {u, v} in increasing key (-W_uv, min(u,v), max(u,v)), where W_uv is
// the heavier of |a_uv| and |a_vu| (the first occurrence of the pair in the
// sorted edge list).  Same rounds of locally dominant edges, for this key:
// every undecided vertex points to its best edge to an undecided neighbour;
// mutual pointers match; a vertex with no undecided neighbour is a
// singleton.  A pointer changes only when a neighbour is decided, so each
// round recomputes the pointers of the vertices next to the previous round's
// decisions ("dirty"), then (after a launch boundary) matches mutual pairs.
// ---------------------------------------------------------------------------
namespace {
struct EdgeKey {
    double w;
    int lo, hi;
    __device__ __forceinline__ bool better(const EdgeKey& o) const {  // smaller key
        if (w != o.w) return w > o.w;
        if (lo != o.lo) return lo < o.lo;
        return hi < o.hi;
    }
};
}  // namespace

__global__ __launch_bounds__(BS) void k_ehem_init(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                                                  const double* __restrict__ v, double* __restrict__ wsym,
                                                  int* __restrict__ dec, int* __restrict__ mate,
                                                  int* __restrict__ ptr, int* __restrict__ stamp,
                                                  int* __restrict__ wl0, int* cnt, int* err) {
    const int u = blockIdx.x * BS + threadIdx.x;
    if (u >= n) return;
    dec[u] = kUndecided;
    mate[u] = -1;
    ptr[u] = -1;
    stamp[u] = -1;
    wl0[u] = u;  // every vertex starts dirty
    if (u == 0) cnt[0] = n;
    bool bad = false;
    for (int e = rp[u]; e < rp[u + 1]; ++e) {
        const int x = ci[e];
        double w = 0.0;
        if (x != u) {
            const int pos = find_col(ci, rp[x], rp[x + 1], u);
            if (pos < 0) bad = true;
            const double back = pos >= 0 ? fabs(v[pos]) : 0.0;
            const double fwd = fabs(v[e]);
            w = fwd > back ? fwd : back;
        }
        wsym[e] = w;
    }
    if (bad) atomicOr(err, ERR_NONSYM);
}

// pointer of each dirty undecided vertex (state at the start of the round)
__global__ __launch_bounds__(BS) void k_ehem_point(int r, const int* __restrict__ rp, const int* __restrict__ ci,
                                                   const double* __restrict__ wsym, const int* __restrict__ dec,
                                                   int* __restrict__ ptr, const int* __restrict__ win, int* cnt,
                                                   int slot_in, int zero_w) {
    if (blockIdx.x == 0 && threadIdx.x == 0) cnt[zero_w] = 0;
    const int m = cnt[slot_in];
    if (m > 0 && blockIdx.x == 0 && threadIdx.x == 0) cnt[6] = r + 1;  // rounds with work
    for (int idx = blockIdx.x * BS + threadIdx.x; idx < m; idx += gridDim.x * BS) {
        const int u = win[idx];
        if (dec[u] != kUndecided) continue;
        EdgeKey best{-1.0, 0, 0};
        int bv = -1;
        for (int e = rp[u]; e < rp[u + 1]; ++e) {
            const int x = ci[e];
            const double w = wsym[e];
            if (x == u || w == 0.0 || dec[x] != kUndecided) continue;
            const EdgeKey k{w, min(u, x), max(u, x)};
            if (bv < 0 || k.better(best)) {
                best = k;
                bv = x;
            }
        }
        ptr[u] = bv;
    }
}

// mutual pointers match; the undecided neighbours of each decision are the
// next round's dirty vertices (marked once per round through the stamps)
__global__ __launch_bounds__(BS) void k_ehem_match(int r, const int* __restrict__ rp, const int* __restrict__ ci,
                                                   const double* __restrict__ wsym, int* __restrict__ dec,
                                                   int* __restrict__ mate, const int* __restrict__ ptr,
                                                   int* __restrict__ stamp, const int* __restrict__ win,
                                                   int* __restrict__ wout, int* cnt, int slot_in, int slot_out) {
    const int m = cnt[slot_in];
    for (int idx = blockIdx.x * BS + threadIdx.x; idx < m; idx += gridDim.x * BS) {
        const int u = win[idx];
        if (dec[u] != kUndecided) continue;
        const int v = ptr[u];
        if (v < 0) {  // no undecided neighbour: unaggregated singleton
            dec[u] = r;
            mate[u] = -1;
            continue;
        }
        if (ptr[v] != u) continue;
        // matched (found by u, and by v too if v is dirty: identical writes)
        dec[u] = r;
        dec[v] = r;
        mate[u] = v;
        mate[v] = u;
        for (int q = 0; q < 2; ++q) {
            const int x = q == 0 ? u : v;
            for (int e = rp[x]; e < rp[x + 1]; ++e) {
                const int y = ci[e];
                if (y == x || wsym[e] == 0.0) continue;
                if (atomicExch(&stamp[y], r) != r) wout[atomicAdd(&cnt[slot_out], 1)] = y;
            }
        }
    }
}

void launch_ehem_init(int n, const int* rp, const int* ci, const double* v, HemWork& w, hipStream_t s) {
    hipLaunchKernelGGL(k_ehem_init, dim3(blocks_for(n)), dim3(BS), 0, s, n, rp, ci, v, w.wsym, w.dec, w.mate,
                       w.ptr, w.lcnt, w.wl[0], w.cnt, w.err);
}

void launch_ehem_round(int r, int n, const int* rp, const int* ci, HemWork& w, hipStream_t s) {
    const int g = blocks_for(n, BS, 4 * w.round_grid);
    hipLaunchKernelGGL(k_ehem_point, dim3(g), dim3(BS), 0, s, r, rp, ci, w.wsym, w.dec, w.ptr, w.wl[r & 1], w.cnt,
                       r % 3, (r + 2) % 3);
    hipLaunchKernelGGL(k_ehem_match, dim3(g), dim3(BS), 0, s, r, rp, ci, w.wsym, w.dec, w.mate, w.ptr, w.lcnt,
                       w.wl[r & 1], w.wl[(r + 1) & 1], w.cnt, r % 3, (r + 1) % 3);
}

// ---------------------------------------------------------------------------
// Matching from the last index (Section 2.1.1): vertices visited downward and
// row entries scanned downward, ties to the highest index.  Renumbering
// i -> n-1-i turns this into the upward pass, so it runs the kernels above on
// the mirrored matrix and maps the pairs back.  Mirroring reverses the order
// of the rows and, with it, of the entries inside each row: the column and
// value arrays are read backwards as a whole and the columns stay ascending.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(BS) void k_mirror_csr(int n, int64_t nnz, const int* __restrict__ rp,
                                                   const int* __restrict__ ci, const double* __restrict__ v,
                                                   int* __restrict__ mrp, int* __restrict__ mci,
                                                   double* __restrict__ mv) {
    const int64_t e = (int64_t)blockIdx.x * BS + threadIdx.x;
    if (e < nnz) {
        mci[e] = n - 1 - ci[nnz - 1 - e];
        mv[e] = v[nnz - 1 - e];
    }
    if (e <= n) mrp[e] = (int)(nnz - rp[n - e]);
}

__global__ __launch_bounds__(BS) void k_unmirror_mate(int n, const int* __restrict__ mr, int* __restrict__ mate) {
    const int i = blockIdx.x * BS + threadIdx.x;
    if (i >= n) return;
    const int m = mr[n - 1 - i];
    mate[i] = m < 0 ? -1 : n - 1 - m;
}

void launch_mirror_csr(int n, int64_t nnz, const int* rp, const int* ci, const double* v, int* mrp, int* mci,
                       double* mv, hipStream_t s) {
    const int64_t work = nnz > (int64_t)n + 1 ? nnz : (int64_t)n + 1;
    hipLaunchKernelGGL(k_mirror_csr, dim3(blocks_for(work)), dim3(BS), 0, s, n, nnz, rp, ci, v, mrp, mci, mv);
}

void launch_unmirror_mate(int n, const int* mr, int* mate, hipStream_t s) {
    hipLaunchKernelGGL(k_unmirror_mate, dim3(blocks_for(n)), dim3(BS), 0, s, n, mr, mate);
}

// Record entries of a pass, by its average row: rows of up to 7.5 entries (the
// 5- and 7-point operators and what regular aggregates make of them) have 2 or
// 3 higher neighbours; the coarse operators of irregular aggregates have up to
// a dozen at 14 entries a row and up to about 30 at 20.  A longer list goes on
// in the row, which costs a few microseconds each time it is needed.
static int hem_record(int n, int64_t nnz, size_t room) {
    const double avg = (double)nnz / n;
    const int r = avg <= 7.5 ? 4 : avg <= 14.0 ? 16 : 32;
    return r == 32 && (size_t)n * 32 > room ? 16 : r;
}

constexpr int kLongRows = 32;  // entries a row on average: above, passes take tiles of
constexpr int kLongTile = 8;   // this many rows (see launch_hem_tile)

// Room for the records of every pass of a setup (a later pass has fewer rows, but
// may have longer ones), and for the mirror images of rows that records do not
// hold: a first pass of short rows has next to none.
size_t hem_rec_ints(int n, int64_t nnz) { return (nnz > 14 * (int64_t)n ? 32 : 16) * (size_t)n; }
size_t hem_ent_ints(int n, int64_t nnz) { return (size_t)(2 * nnz <= 15 * (int64_t)n ? nnz / 2 : nnz); }

void launch_hem_init(int n, int64_t nnz, const int* rp, const int* ci, const double* v, HemWork& w, hipStream_t s) {
    w.side = hem_record(n, nnz, w.rec_ints);
    const bool thread = w.side == 4 && n > kInitThread;
    w.long_rows = nnz > kLongRows * (int64_t)n;
    w.mirrors = !thread && (size_t)nnz <= w.ent_ints;
    int* const ent = w.mirrors ? w.ent : nullptr;
#define CALL(K, grid, ...)                                                                                       \
    hipLaunchKernelGGL(K, dim3(grid), dim3(BS), 0, s, n, rp, ci, v, w.rec, w.deg, w.gw, w.xw, w.mate, w.cnt, w.err, \
                       ##__VA_ARGS__)
    if (w.side == 32) CALL((k_hem_init_group<32, 32>), blocks_for(n, BS / 32, kInitBlocks), ent);
    else if (w.side == 16) CALL((k_hem_init_group<16, 16>), blocks_for(n, BS / 16, kInitBlocks), ent);
    else if (!thread) CALL((k_hem_init_group<4, 16>), blocks_for(n, BS / 16, kInitBlocks), ent);
    else CALL(k_hem_init, blocks_for(n));
#undef CALL
}

// Workgroup sizes.  Larger tiles have fewer steps across tiles (3 to 4 us
// against about 1 us inside one) but more waves that share a compute unit's
// issue slots.  Measured, pass times with workgroups of 1024 / 512 / 256:
//   short rows, 2,097,152 rows (128^3)           2.20 / 1.85 / 2.35 ms
//   short rows, 442,368 rows                     0.50 / 0.43 / 0.54 ms
//   long rows, 512,715 rows of 13.4 entries      2.05 / 1.71 / 1.52 ms
//   long rows, 16,533 rows of 18.6 entries       0.86 / 0.83 / 0.75 ms
//   long rows, 4,440 rows of 18.8 entries        0.47 / 0.51 / 0.54 ms
constexpr int kFewRows = 10000;  // long rows: up to here the large tiles win
// Rows longer than that are mostly wide, or have neighbours that are, and are
// then read again by a whole wave, one vertex after the other: a wave takes few
// vertices.  Their words are in memory anyhow, so little is lost between tiles.
// Pass times with tiles of 2 / 8 / 16 / 64 rows / as many as a workgroup takes:
//   10,978 rows of 104 entries     1.65 / 2.00 / 2.43 / 4.14 / 4.40 ms
//    2,748 rows of 81 entries      0.85 / 1.08 / 1.31 / 2.15 / 3.76 ms
//    5,488 rows of 39 entries      0.32 / 0.26 / 0.27 / 0.33 / 0.34 ms
//    2,744 rows of 23 entries      0.23 / 0.17 / 0.20 / 0.28 / 0.28 ms
//       89 rows of 25 entries      0.08 / 0.08 / 0.09 / 0.10 / 0.10 ms
//      686 rows of 21 entries      0.13 / 0.11 / 0.11 / 0.12 / 0.08 ms

void launch_hem_tile(int n, const int* rp, const int* ci, const double* v, HemWork& w, long long tmo,
                     hipStream_t s) {
    const HemState S{n, rp, ci, v, w.rec, w.deg, w.mirrors ? w.ent : nullptr, w.gw, w.xw, w.mate};
    const bool long_rows = w.long_rows && w.side == 32;
#define CALL(R, NT)                                                                                               \
    {                                                                                                             \
        const int tm = long_rows ? kLongTile : NT - 2 * kWave;                                                    \
        const int rows = w.tile_rows > 0 && w.tile_rows < tm ? w.tile_rows : tm;                                  \
        hipLaunchKernelGGL((k_hem_tile<R, NT>), dim3((unsigned)(((int64_t)n + rows - 1) / rows)), dim3(NT), 0, s, \
                           S, rows, w.cnt, w.err, tmo);                                                           \
    }
    if (w.side == 4) CALL(4, 512)
    else if (w.side == 16 && n > kFewRows) CALL(16, 256)
    else if (w.side == 16) CALL(16, 1024)
    else if (n > kFewRows || long_rows) CALL(32, 256)
    else CALL(32, 1024)
#undef CALL
}

}  // namespace amg
