// Internal interfaces between the host orchestration (amg_api.hip) and the
// kernel launchers (k_setup.hip, k_solve.hip).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace amg {

// Device error bits raised by validation and setup kernels.
enum : int {
    ERR_STRUCT = 1,      // bad row_ptr / column index / column order
    ERR_NONFINITE = 2,   // NaN or Inf value
    ERR_DIAG = 4,        // missing or zero diagonal
    ERR_NONSYM = 8,      // pattern not structurally symmetric
    ERR_SINGULAR = 16,   // the coarsest matrix has a zero pivot
};

constexpr int kUndecided = 0x3fffffff;  // round stamp of an undecided vertex
constexpr int kDenseMaxRows = 4096;     // largest coarsest level (explicit inverse)

// Lanes per CSR row used by the level kernels (a power of two, 1..16).
int pick_lanes_per_row(double avg_row_len);

// ---- setup kernels (k_setup.hip) ------------------------------------------
// Column codes (amg_stream.hpp) of the rows of a validated matrix, one record
// per 64 rows; *uncoded += the slices that need more than the record holds.
struct SliceCode;
size_t slice_code_bytes(int n);
void launch_code_slices(int n, const int* rp, const int* ci, SliceCode* code, int* uncoded, hipStream_t s);
void launch_validate(int n, int64_t nnz, const int* rp, const int* ci, const double* v, double* dinv, int* err,
                     hipStream_t s);
void launch_dinv(int n, const int* rp, const int* ci, const double* v, double* dinv, int* err, hipStream_t s);

// Buffers of a matching pass (k_hem.hip).
struct HemWork {
    int* rec;         // records of 4, 16 or 32 entries a vertex
    size_t rec_ints;  // room for them
    int* ent;         // mirror images of the entries of rows that their records do not hold
    size_t ent_ints;  // room for them
    bool mirrors = false;  // the current pass has them
    bool long_rows = false;  // the current pass takes small tiles
    int2* deg;        // [n] lower entries (or extension offset) and higher edge-neighbours
    unsigned* gw;     // [n] a vertex's word as set by other tiles
    unsigned* xw;     // [hem_ext_words(nnz)] extension words of rows with many lower entries
    int* mate;        // [n] partner or -1
    int* cnt;         // [8] tiles started, extension words, symmetry check, sweeps, time limit
    int* err;
    int side = 4;            // entries of the current pass's records
    int tile_rows = 0;       // rows per tile, at most what a workgroup takes (0: that many)
    // edge-based matching
    int* dec;         // [n] round in which the vertex was decided
    int* lcnt;        // [n] round marks
    int* wl[2];       // [n] worklists (ping-pong)
    double* wsym = nullptr;  // [nnz] heavier of |a_uv|, |a_vu| (0 on the diagonal)
    int* ptr = nullptr;      // [n] best undecided neighbour
    int round_grid = 96;     // blocks of a round's launches
};
// Extension words of a pass: a row of more than 31 lower entries takes one word
// and one per 32 of them (at most 3/32 of their number).
inline size_t hem_ext_words(int64_t nnz) { return (size_t)(nnz / 10 + 64); }
size_t hem_rec_ints(int n, int64_t nnz);
size_t hem_ent_ints(int n, int64_t nnz);
// Node-based pass (w.cnt must be zeroed before the initialisation): all tiles
// in one launch.  cnt[7] != 0 afterwards: it did not finish within tmo
// wall-clock ticks and must be repeated.
void launch_hem_init(int n, int64_t nnz, const int* rp, const int* ci, const double* v, HemWork& w, hipStream_t s);
void launch_hem_tile(int n, const int* rp, const int* ci, const double* v, HemWork& w, long long tmo, hipStream_t s);
// Edge-based matching (Algorithm 3): initialisation (every vertex dirty, the
// count in cnt[0]; w.lcnt serves as the per-round marks) and one round (two
// launches).  w.cnt must be zeroed before the initialisation.
void launch_ehem_init(int n, const int* rp, const int* ci, const double* v, HemWork& w, hipStream_t s);
void launch_ehem_round(int r, int n, const int* rp, const int* ci, HemWork& w, hipStream_t s);

size_t scan_tmp_ints(int n);  // scratch of the two prefix sums below
// A thread's pinned words.  What a pass hands to the host has a place of its own:
// the host takes it to have arrived when the sequence word has its value, which
// no read-back may store there meanwhile.
constexpr int kPinnedWords = 64;
constexpr int kReadWords = 32;                 // read-backs: the first words
constexpr int kRoundWords = kReadWords, kRounds = 2;  // worklist sizes of the edge-based rounds
constexpr int kPassWords = 40;                 // a pass's words
constexpr int kPassSeq = 12;                   // the sequence word among them, the last one
static_assert(kRoundWords + kRounds <= kPassWords && kPassWords + kPassSeq < kPinnedWords, "places of their own");
struct PassWords {
    int* out;        // mapped host memory: cnt[0 .. 7], *nc, the entry count, *err, *novf, seq
    int* cnt;        // cleared after
    const int* nc;
    const int* err;
    const int* novf;
    int seq;
};
// From the mates: agg[v] = id of v's aggregate, lead[id] = smaller vertex of
// the aggregate, the coarse row count; *novf = 0.
void launch_numbering(int n, const int* mate, int* agg, int* lead, int* nc, int* novf, int* tmp, hipStream_t s);
// crp[0 .. n] = exclusive sums of the counts, and the pass's words.
void launch_offsets(int n, const int* rowcnt, int* crp, const PassWords& w, int* tmp, hipStream_t s);
// Galerkin product of one matching pass (aggregates of size <= 2).
// n, nnz: rows and entries of the fine operator
void launch_rap_count(int nmax, int64_t nnz, const int* ncp, const int* lead, const int* mate, const int* rp,
                      const int* ci, const int* agg, int* rowcnt, int* ovf, int* novf, hipStream_t s);
void launch_rap_count_slow(int nc, const int* ovf, const int* novf, const int* lead, const int* mate, const int* rp,
                           const int* ci, const int* agg, int* rowcnt, hipStream_t s);
void launch_rap_fill(int nc, int n, int64_t nnz, const int* lead, const int* mate, const int* rp, const int* ci,
                     const double* v, const int* agg, const int* crp, int* cci, double* cv, hipStream_t s);
void launch_rap_fill_slow(int nc, const int* ovf, const int* novf, const int* lead, const int* mate, const int* rp,
                          const int* ci, const double* v, const int* agg, const int* crp, int* cci, double* cv,
                          hipStream_t s);

// Matching from the last index: the mirrored matrix (i -> n-1-i) and the map of
// its pairs back to the original numbering.
void launch_mirror_csr(int n, int64_t nnz, const int* rp, const int* ci, const double* v, int* mrp, int* mci,
                       double* mv, hipStream_t s);
void launch_unmirror_mate(int n, const int* mr, int* mate, hipStream_t s);

void launch_compose(int n, const int* agg1, const int* agg2, int* out, hipStream_t s);
// Member lists (ascending fine rows, -1 padded) of the level's coarse rows.
void launch_members(int nc, const int* lead2, const int* mate2, const int* lead1, const int* mate1, int4* mem,
                    hipStream_t s);

// Systems stored one after another in a level: out[2j] = agg[off[j]],
// out[2j+1] = crp[out[2j]] (coarse row and entry where system j starts).
void launch_seg_starts(int m, const int* off, const int* agg, const int* crp, int* out, hipStream_t s);

// ---- coarsest inverse (k_dense.hip) -----------------------------------------
// One system: n <= kDenseMaxRows CSR rows; col_add shifts the stored columns (a
// diagonal block of a larger matrix; entries outside the block are skipped).
// ainv_t receives the inverse column-major; err |= ERR_SINGULAR on a zero pivot.
struct DenseJob {
    int n;
    int col_add;
    const int* rp;
    const int* ci;
    const double* v;
    double* ainv_t;
    int* err;
};
constexpr int kDenseSmall = 128;  // systems up to this size take one workgroup and no workspace
// Systems of at most nmax <= kDenseSmall rows, one workgroup each: the `count`
// jobs at `many` (device), or `one` when that is null.
void launch_dense_small(const DenseJob& one, const DenseJob* many, int count, int nmax, hipStream_t s);
// Any size; work: dense_work_doubles(n) doubles.
size_t dense_work_doubles(int n);
void launch_dense_inverse(const DenseJob& J, double* work, hipStream_t s);

// ---- solve kernels (k_solve.hip) --------------------------------------------
struct LevelView {
    int n;
    int nnz;
    const int* rp;
    const int* ci;
    const double* v;
    const double* dinv;
    const int* agg;   // [n] aggregate on level k+1
    const int4* mem;  // [n_{k+1}] members of coarse rows (for k < L)
    int lpr;          // lanes per row
    const SliceCode* code;  // column codes of its rows, or null
};

struct Reducer {
    double* part;     // [2 * kRedBlocks] per-block partial sums
    double* S;        // scalar slots
};

// A coarse level's finished value zc of row i becomes the finer level's
// prolongated iterate on i's members m: xpf[m] = w gf[m] + zc.
template <class T>
struct ScatterT {
    const int4* __restrict__ mem;
    const T* __restrict__ gf;
    T* __restrict__ xpf;
    T w;
    __device__ __forceinline__ void operator()(int i, T zc) const {
        const int4 m = mem[i];
        xpf[m.x] = w * gf[m.x] + zc;
        if (m.y >= 0) xpf[m.y] = w * gf[m.y] + zc;
        if (m.z >= 0) xpf[m.z] = w * gf[m.z] + zc;
        if (m.w >= 0) xpf[m.w] = w * gf[m.w] + zc;
    }
};

// V-cycle view of a level with values of type T (double, or the float copy).
template <class T>
struct VLevel {
    int n;
    const int* rp;
    const int* ci;
    const T* v;
    const T* dinv;
    const int4* mem;  // members of level k+1 rows
    int lpr;
    int rb = 256;     // rows per block of the CSR-stream kernels: 128, 256 or 512
    const SliceCode* code = nullptr;  // column codes of its rows: the CSR-stream kernels then read those
    int order = 0;    // CSR-stream kernels: 4 or 8 adds as the lane-group kernels with that many lanes
};

// ---- V-cycle kernels (k_vcycle.hip), T = double or float -------------------
// Every level keeps g = D^{-1} f next to its right-hand side f; the kernel
// that produces f also writes g.  Large levels (CSR-stream): r = f - w A g,
// then f_c = P^T r and g_c; postsmoothing from the prolongated iterate xp:
// z = xp + w (g - D^{-1} A xp), with (f, z) reduced into `slot` when R is
// given and z scattered into the finer level's xp when sc is given.
template <class T, class TIN>
void vc_stream_resid(const VLevel<T>& L, const TIN* f, const T* g, T w, T* r, hipStream_t s);
template <class T>
void vc_restrict(int nc, const int4* mem, const T* r, const T* dinv_c, T* fc, T* gc, hipStream_t s);
// slot == kPartialsOnly: the (f, z) partials stay in R->part (at most
// kFusedParts blocks) for a consumer kernel to add; returns their number (0
// when no partials are left).
template <class T, class TOUT>
int vc_stream_post(const VLevel<T>& L, const T* xp, const T* g, T w, TOUT* z, const double* f, const Reducer* R,
                   int slot, const ScatterT<T>* sc, hipStream_t s, hipEvent_t t0 = nullptr,
                   hipEvent_t t1 = nullptr);  // t0/t1: recorded at the start/end of the main kernel
// Small levels: the same operations with the restriction fused.
template <class T, class TIN>
void vc_resid_restrict(const VLevel<T>& L, int nc, const TIN* f, const T* g, T w, const T* dinv_c, T* fc, T* gc,
                       hipStream_t s);
template <class T, class TOUT>
void vc_prolong_post(const VLevel<T>& L, const T* xp, const T* g, T w, TOUT* z, const ScatterT<T>* sc,
                     hipStream_t s);
// The same two on level 0 for a right-hand side whose g = D^{-1} f does not
// exist yet: formed where it is read (in double, rounded to T), stored in g.
template <class T>
void vc_stream_resid_first(const VLevel<T>& L, const double* f, const double* dinv, T w, T* r, T* g, hipStream_t s);
template <class T>
void vc_resid_restrict_first(const VLevel<T>& L, int nc, const double* f, const double* dinv, T w, const T* dinv_c,
                             T* fc, T* gc, T* g, hipStream_t s);
// g = D^{-1} f (computed in double, stored as T)
template <class T>
void vc_scale_dinv(int n, const double* dinv, const double* f, T* g, hipStream_t s);
// Coarsest level x = A_L^{-1} f in double (explicit inverse, column-major).
template <class T, class TIN, class TOUT>
void vc_dense_apply(int n, const double* ainv_t, const TIN* f, TOUT* x, const ScatterT<T>* sc, hipStream_t s);

// The small levels in one workgroup (k_tail.hip).  Level l = 0 .. nl - 1
// smooths, level nl is the coarsest; offsets are bytes in LDS, where the
// packed block of the levels' operators comes first, headed by their records.
constexpr int kTailLevels = 16;
// Most coarsest rows: one CU reads the inverse, 8 bytes a square.  With 207 rows a
// V-cycle on 91 x 75 x 64 rows takes 99.6 us (102.3 without a tail), with 349 one on
// 160^3 298 (282).
constexpr int kTailDense = 256;
constexpr uint16_t kTailNone = 0xffff;   // no such member
struct alignas(16) TailLevel {
    int n, nc;                      // rows, rows of the next level
    int v, dinv, ci, rec;           // operator, its rows by member of the next level's rows
    int g, a;                       // D^{-1} f, then z; f, then xp
    int cg, ca, cdinv;              // g, a and dinv of the next level
    int lpr_log;                    // log2 of the lanes per row (1 or 2)
    int pad[4];
};
static_assert(sizeof(TailLevel) == 64, "four 16-byte words");
template <class T>
struct TailArgs {
    const uint4* blob;
    const double* ainv;  // coarsest inverse, column-major
    const T* f;          // right-hand side of level 0 and g = D^{-1} f
    const T* g;
    T w;
    int words;           // 16-byte words of the block
    int nl, n0, m;       // smoothing levels; finest and coarsest rows
    int g0, a0, gm, am;  // their vectors
    int part;            // partial sums of the coarsest solve
};
template <class T>
struct TailJob {
    TailArgs<T> a;
    ScatterT<T> sc;
};
// A level's arrays; the `add`s give the system's own numbering.  v or dinv
// null: rounded from the double ones.
template <class T>
struct TailSrc {
    const int* rp;
    const int* ci;
    const T* v;
    const T* dinv;
    const int4* mem;
    int nnz;
    int rp_add, ci_add, mem_add;
    const double* v64;
    const double* dinv64;
};
template <class T>
struct TailPack {
    char* blob;
    int nl;
    TailSrc<T> src[kTailLevels];
    TailLevel lev[kTailLevels];
};
// n[0 .. nl], nnz and lanes per row [0 .. nl - 1]: the LDS bytes of the cycle on these levels, or
// 0 when it does not fit; fills lev[0 .. nl - 1] and A (not its pointers).  lpr
// null: for the CSR-stream kernels' order.
template <class T>
int tail_layout(const int* n, const int64_t* nnz, const int* lpr, int nl, TailArgs<T>& A, TailLevel* lev);
template <class T>
void launch_tail_pack(const TailPack<T>& K, int nl, hipStream_t s);
template <class T>
void vc_tail(const TailArgs<T>& A, int lds, const ScatterT<T>& sc, hipStream_t s);
// Many systems at once: jobs and packs in device memory, nl the most levels of
// a system.
template <class T>
void launch_tail_packs(const TailPack<T>* K, int count, int nl, hipStream_t s);
template <class T>
void vc_tails(const TailJob<T>* jobs, int count, int lds, hipStream_t s);
bool tail_prepare();  // whether the device takes the tail kernels

// S[slot0] (and S[slot1] when nv = 2) = fixed-order sums of the partials.
void launch_cast_f32(int64_t n, const double* a, float* b, hipStream_t s);
void launch_finish(int nparts, int nv, const Reducer& R, int slot0, int slot1, hipStream_t s);

// General smoothing path.
void launch_jacobi_zero(int n, const double* dinv, const double* f, double w, double* x, hipStream_t s);
void launch_jacobi(const LevelView& L, const double* f, const double* x, double w, double* xo, hipStream_t s);
void launch_resid_restrict_x(const LevelView& L, int nc, const double* f, const double* x, double* fc,
                             hipStream_t s);
void launch_prolong_add(int n, const int* agg, const double* e, double* x, hipStream_t s);

// Krylov vector kernels.  Slots index Reducer::S.
// r = b - A x, (r, r); gout (may be null) receives D^{-1} r, as float when g32.
void launch_residual(const LevelView& A, const double* b, const double* x, double* r, void* gout, bool g32,
                     const Reducer& R, int slot_rr, hipStream_t s);
void launch_dot(int n, const double* a, const double* b, const Reducer& R, int slot, hipStream_t s);
void launch_spmv_dot(const LevelView& A, const double* p, double* q, const double* d, const Reducer& R, int slot,
                     hipStream_t s);
// q = A p with the block partials of (d, q) left in part (at most
// kFusedParts blocks); returns their number.
int launch_spmv_dot_parts(const LevelView& A, const double* p, double* q, const double* d, double* part,
                          hipStream_t s);
void launch_spmv_dot2(const LevelView& A, const double* p, double* t, const double* sv, const Reducer& R, int slot_tt,
                      int slot_ts, hipStream_t s);
// pq_part (non-null): the update adds the pq_np partials of (p, q) itself
// (block 0 stores the sum in slot_pq) and leaves the partials of (r, r) in
// rr_part (at most kFusedParts blocks; *rr_np receives their number) instead
// of finishing them into slot_rr.
void launch_cg_update(int n, double* x, double* r, const double* p, const double* q, const double* dinv, void* gout,
                      bool g32, const Reducer& R, int slot_rho, int slot_pq, int slot_rr, hipStream_t s,
                      const double* pq_part = nullptr, int pq_np = 0, double* rr_part = nullptr, int* rr_np = nullptr);
// Sh/nsh: optional host memory mapped into the device that receives the
// first nsh scalar slots (nsh <= 256).  new_part (non-null): the kernel adds
// the new_np partials of the new (r, z) itself (block 0 stores the sum in
// slot_new).  rr_part (non-null): block 0 adds the rr_np partials of (r, r)
// into slot_rr.  hseq (non-null, with Sh): after the slots, the word hseq
// (mapped host memory too) receives seq, so the host can wait for the slots
// by watching that word.
void launch_cg_dir(int n, const double* z, const double* p, double* pn, double* S, int slot_new, int slot_old,
                   hipStream_t s, double* Sh = nullptr, int nsh = 0, const double* new_part = nullptr, int new_np = 0,
                   const double* rr_part = nullptr, int rr_np = 0, int slot_rr = 0, unsigned long long* hseq = nullptr,
                   unsigned long long seq = 0);
void launch_bicg_s(int n, const double* r, const double* v, double* sv, const double* S, int slot_rho, int slot_rv,
                   hipStream_t s);
void launch_bicg_update(int n, double* x, double* r, const double* pt, const double* st, const double* sv,
                        const double* t, const double* rb, const Reducer& R, int slot_rho, int slot_rv, int slot_tt,
                        int slot_ts, int slot_rr, int slot_rhonew, hipStream_t s);
// Sh/nsh/hseq/seq: the slot hand-over into mapped host memory (see the PCG
// direction kernel); null leaves it out.
void launch_bicg_dir(int n, const double* r, const double* p, const double* v, double* pn, const double* S,
                     int slot_rho, int slot_rv, int slot_tt, int slot_ts, int slot_rhonew, hipStream_t s,
                     double* Sh = nullptr, int nsh = 0, unsigned long long* hseq = nullptr,
                     unsigned long long seq = 0);
void launch_scale_zero(int n, double* x, hipStream_t s);
void launch_add(int n, double* x, const double* z, hipStream_t s);
// err |= ERR_NONFINITE if any entry of a or b is NaN or Inf.
void launch_check_finite(int n, const double* a, const double* b, int* err, hipStream_t s);

constexpr int kRedBlocks = 65536;  // max blocks (partials) of a reduction kernel
// Reductions whose consumer kernel adds the partials itself use at most this
// many blocks (each consumer block reads them all).
constexpr int kFusedParts = 2048;
// Partial regions of the PCG iteration inside Reducer::part (each holds up to
// kFusedParts): (p, q) of the SpMV, (r, r) of the update, (r, z) of the
// level-0 postsmoothing.
constexpr int kPartPQ = 0, kPartRR = 4096, kPartRZ = 8192;
constexpr int kPartialsOnly = -2;  // slot value: leave the block partials, no finish kernel

// ---- batched solves (k_batch.hip) -------------------------------------------
// Systems ("segments") stored one after another.  blk[b] = (segment, first
// row) of reduction block b (256 rows, never crossing a segment end);
// seg_end[s] = one past the segment's last row; mask[s] != 0 selects the
// segments a launch works on.  Scalars: S[s * kBatchSlots + slot].
constexpr int kBatchSlots = 8;
struct BatchTab {
    const int2* blk;
    const int* seg_end;
    const int* mask;
};
// Coarsest solve of one segment: x = A_L^{-1} f on n rows (f, x already
// offset to the segment), each result scattered to the finer level's rows
// through sc at index row0 + i.
template <class T>
struct BDense {
    int n;
    int row0;
    const double* ainv_t;
    const T* f;
    T* x;
    ScatterT<T> sc;
};
// One copy of a batch assembly: kind 0 int32 (+add), 1 double, 2 float,
// 3 int4 member lists (+add on the members present), 4 double rounded to
// float.
struct GatherPiece {
    const void* src;
    void* dst;
    int64_t count;
    int add;
    int kind;
};
int gather_chunk();  // elements per block of launch_gather

void launch_bspmv_dot(int nblk, const BatchTab& T, const int* rp, const int* ci, const double* v, const double* p,
                      double* q, const double* d, double* part, hipStream_t s);
void launch_bresidual(int nblk, const BatchTab& T, const int* rp, const int* ci, const double* v, const double* x,
                      const double* b, double* r, const double* dinv, void* g, bool g32, double* part,
                      hipStream_t s);
void launch_bdot(int nblk, const BatchTab& T, const double* a, const double* c, double* part, hipStream_t s);
void launch_bfinish(int nseg, const int* seg_blk, const int* mask, const double* part, double* S, int slot_k,
                    hipStream_t s);
// seg_blk and pq_part (or null: the slot holds it): the kernel adds the
// partials of (p, q) itself and stores the sum in slot_pq
void launch_bcg_update(int nblk, const BatchTab& T, double* x, double* r, const double* p, const double* q,
                       const double* dinv, void* g, bool g32, double* part, double* S, int slot_rho, int slot_pq,
                       const int* seg_blk, const double* pq_part, hipStream_t s);
// with rz_part: the kernel adds the partials of (r, z) into slot_new and those
// of (r, r) into slot_rr
void launch_bcg_dir(int nblk, const BatchTab& T, const double* z, const double* p, double* pn, double* S,
                    int slot_new, int slot_old, hipStream_t s, const int* seg_blk = nullptr,
                    const double* rz_part = nullptr, const double* rr_part = nullptr, int slot_rr = 0);
void launch_bzero(int nblk, const BatchTab& T, double* x, hipStream_t s);
// Algorithm 5 over a batch (two-sum kernels write their second partials at part + nblk).
void launch_bbicg_s(int nblk, const BatchTab& T, const double* r, const double* v, double* sv, const double* S,
                    int slot_rho, int slot_rv, hipStream_t s);
void launch_bspmv_dot2(int nblk, const BatchTab& T, const int* rp, const int* ci, const double* v, const double* st,
                       double* t, const double* sv, double* part, hipStream_t s);
void launch_bbicg_update(int nblk, const BatchTab& T, double* x, double* r, const double* pt, const double* st,
                         const double* sv, const double* t, const double* rb, double* part, const double* S,
                         int slot_rho, int slot_rv, int slot_tt, int slot_ts, hipStream_t s);
void launch_bbicg_dir(int nblk, const BatchTab& T, const double* r, const double* p, const double* v, double* pn,
                      const double* S, int slot_rho, int slot_rv, int slot_tt, int slot_ts, int slot_rhonew,
                      hipStream_t s);
template <class T>
void launch_bdense(int nblk, const BDense<T>* dd, const int2* tab, hipStream_t s);
void launch_gather(int nblk, const GatherPiece* pcs, const int2* tab, hipStream_t s);

}  // namespace amg
