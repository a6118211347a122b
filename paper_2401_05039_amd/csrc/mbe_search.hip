// Depth-first MBEA search on gfx950 (wave64).
//
// What is computed: the maximal bicliques of Algorithm 1 (MBEA, section II-B), in the
// library's letters: the candidate x joins the growing set L (candidate side C), the
// shrinking set R (other side O) becomes R' = R n N(x), the maximality check fails when a
// vertex of Q is adjacent to all of R', the expansion moves every candidate of P adjacent
// to all of R' into L', and P' / Q' keep the vertices with 0 < |N(v) n R'| < |R'|.  The
// counts come from reverse scanning (section III-E): walk the vertices of R' and their
// neighbours rather than every candidate's list.  Candidates are taken in ascending count
// (sections II-C and III-E), ties in the order of the parent's list.
//
// How it maps to the hardware (the build's own design, not the paper's CUDA one):
//
//  * Coarse grain (section III-C's first-level subtrees): one workgroup owns one top-level
//    candidate x at a time, claimed from a global atomic counter, largest degree first.
//
//  * Local universe.  Every vertex below x is a 2-hop neighbour of x and every R below x is
//    a subset of N(x).  The workgroup runs the reverse scan over N(x) once and gives each
//    2-hop neighbour v the mask M[v] = N(v) n N(x) over the positions of N(x) (W 64-bit
//    words).  Universe entries are numbered in top-level rank order, so the top-level Q is
//    a prefix.  Below the top level the CSR is never read again.
//
//  * Frames.  A frame is the candidate list of one search node: entry k carries its mask
//    restricted to the frame's R, so a child's R' is simply the candidate's own mask.  When
//    |R| <= 64 the masks are compressed to |R| bits (one word).  Each frame also holds the
//    paper's reverse scan turned into an index: for every bit b of R a row, the position bitmap
//    of the entries with b, and tables of the first candidate with b, their number and the sum
//    of their L-side hash terms.  Q entries are rows only.
//
//  * Nodes.  A candidate at position i with |R'| = 1 (almost every node on power-law
//    graphs) is settled by one lookup: it is maximal exactly when the first entry with its
//    bit is itself, and then L' is every entry with that bit.  The 64 lanes of a wave settle
//    64 such candidates at once, and test 64 candidates (or as many as the row words allow) of
//    |R'| >= 2 for maximality at once.  What is left, the maximal nodes of |R'| >= 2, is
//    expanded by the whole wave: one pass over R''s rows finds L', P' and Q'.
//
//    What bounds the search is the wave's instruction and dependent-access chain per node, not
//    bandwidth (a tenth of HBM).  Measured on the power-law graph of 100,000 x 50,000 vertices
//    and 10^6 edges: tests one node at a time, Q' as list entries with masks and shuffles through
//    the LDS pipe 37.6 ms; the tests 64 at a time, Q' as rows (subsets of R' found by word ANDs
//    when |R'| <= 6) and cross-lane moves on the vector pipe 21.0 ms.  Twelve top-level
//    candidates of a 20,000 x 5,000 graph of 2M edges: 280 -> 68 ms.  (With shared lists read in
//    place and every wave stopping where one runs out of stack 19.4 and 52 ms.)
//
//  * Second level (the paper's k = 2 subtrees): the waves of the workgroup claim the candidates
//    of the top-level node's child list that need a full node, one at a time, from an LDS
//    counter; each wave then runs its own depth-first search on an explicit stack of frames (section III-B's goal: no
//    recursion and no allocation; frames are laid back to back in one preallocated array).
//
// Counts and hashes are commutative u64 sums, so results do not depend on which lane, wave
// or workgroup settled which node.

#include "mbe_internal.h"

namespace mbe {

namespace {

constexpr uint64_t kHashK = 0x9E3779B97F4A7C15ull;
constexpr uint32_t kShared = 0xFFFFFFFFu;  // frame offset meaning "the workgroup's top-level list"
// Ticks of the 100 MHz wall clock.  A top-level list is moved out for others only after its
// workgroup has searched it for 0.3 ms: from then on every claim is an add on one address for all,
// and the others read the list through their own L2 (a die has its own), so lists of short items
// are searched sooner by the eight waves that have them at hand.  A graph of 788 x 540 vertices
// with 19,000 edges takes 1.0 ms when lists move after 60 us, 0.53 ms after 0.3 ms and 0.44 ms
// when none moves; the skewed slice (items of milliseconds) takes 1,470 ms without and the same
// 50 ms with either.
constexpr uint32_t kShareAfter = 30000;
constexpr uint32_t kLongItem = 10000;  // an item of 0.1 ms or more is claimed by itself
constexpr uint32_t kMovedMark = 1u << 30;  // added to the LDS item counter when the list moves
constexpr uint32_t kNone = 0xFFFFFFFFu;
constexpr int kQKeep = 256;      // most incomparable Q' masks a compressed child keeps
// A compressed child's Q' (entries with two or more bits of R') is reduced to its
// inclusion-maximal masks when it has more than this many entries.  The reduction compares every
// entry with the masks kept so far; below the line the AND of a few more row words per check
// costs less.  (Also where the row words of the whole Q' would make the frame larger than one with
// the reduced entries' ids, hash terms and masks, the candidates' ids and tables for 64 bits: that
// was the frame's size before Q' became rows alone, and a caller's memory that held it holds this.
// Reducing wherever it saves a row word took the power-law graph from 19.8 to 20.9 ms.)
constexpr int kQReduce = 256;
// A maximal node's P' positions (stu) stay in the wave's LDS for lists of at most this many
// candidates, in global scratch for longer ones.
constexpr int kStuLds = 256;
static_assert(2 * kStuLds >= 64 * 8, "P' masks of 64 entries fit the second half");
constexpr int kWaveLds = 768 + 8 * kQKeep + 4 * kStuLds + 32;  // LDS bytes per wave besides the histogram
// The fixed-width classes keep a graph's rank bitmap and its popcount prefix in LDS, after the
// waves' regions, when the bitmap has at most this many words (131,072 candidates); larger
// graphs keep them in the workgroup's arena slot.
constexpr int kRankLdsWords = 2048;
__host__ __device__ constexpr size_t rank_lds_bytes(int nwords) {
    return nwords <= kRankLdsWords ? ((size_t)nwords * 12 + 4 + 15) / 16 * 16 : 0;
}

// LDS after the workgroup header: the waves' histograms (4 bytes per bit each), which the
// top-level list build reuses for its tables (16 bytes per bit), hence at least that much.
__host__ __device__ constexpr size_t hist_region_bytes(int bits, int waves) {
    return (size_t)bits * (waves >= 4 ? 4 * (size_t)waves : 16);
}

// SplitMix64 output function (Steele, Lea and Flood, OOPSLA 2014).
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z ^= z >> 30;
    z *= 0xBF58476D1CE4E5B9ull;
    z ^= z >> 27;
    z *= 0x94D049BB133111EBull;
    z ^= z >> 31;
    return z;
}
__device__ __forceinline__ uint64_t hash_u(int32_t a) { return mix64(kHashK * (2ull * (uint64_t)(uint32_t)a + 1ull)); }
__device__ __forceinline__ uint64_t hash_v(int32_t b) { return mix64(kHashK * (2ull * (uint64_t)(uint32_t)b + 2ull)); }
__device__ __forceinline__ uint64_t pair_hash(int c_is_v, uint64_t sL, uint64_t sR) {
    // h(A, B) = mix(sum hu(A) + mix(sum hv(B) + K)); A is the U side.
    return c_is_v ? mix64(sR + mix64(sL + kHashK)) : mix64(sL + mix64(sR + kHashK));
}

__device__ __forceinline__ int lane_id() { return (int)__lane_id(); }

// Wave-uniform values moved to scalar registers (the value of the first active lane; only
// for values every lane holds alike).
__device__ __forceinline__ int32_t uni(int32_t x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ uint32_t uni(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }
__device__ __forceinline__ uint64_t uni(uint64_t x) {
    return ((uint64_t)uni((uint32_t)(x >> 32)) << 32) | (uint64_t)uni((uint32_t)x);
}
// lane 63's value (a wave-wide scan total) in a scalar register
__device__ __forceinline__ int last_lane(int x) { return __builtin_amdgcn_readlane(x, 63); }
__device__ __forceinline__ uint64_t lanes_below() { return (1ull << lane_id()) - 1ull; }

// Cross-lane moves on the vector pipe: DPP within rows of 16 lanes, the row and half swaps
// between them.  (Shuffles through the LDS pipe are a round trip of some 60-100 cycles each,
// six of them in a row for a reduction or a transpose, on the critical path of every node.)
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_mov(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, CTRL, 0xF, 0xF, true);
}

// x of the lane CTRL names in the rows of mask ROWS, 0 elsewhere (shifts bring 0 in)
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_or_zero(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xF, false);
}
// Inclusive scan with a commutative operation whose identity is 0: shifts by 1, 2, 4 and 8
// within each row of 16, then lane 15 of rows 0 and 2 into the next row, lane 31 into the upper
// half.  All 64 lanes are active.
template <typename Op>
__device__ __forceinline__ uint32_t wave_scan32(uint32_t v, Op op) {
    v = op(v, dpp_or_zero<0x111, 0xF>(v));
    v = op(v, dpp_or_zero<0x112, 0xF>(v));
    v = op(v, dpp_or_zero<0x114, 0xF>(v));
    v = op(v, dpp_or_zero<0x118, 0xF>(v));
    v = op(v, dpp_or_zero<0x142, 0xA>(v));
    return op(v, dpp_or_zero<0x143, 0xC>(v));
}
template <int CTRL, int ROWS>
__device__ __forceinline__ uint64_t dpp_or_zero64(uint64_t x) {
    return ((uint64_t)dpp_or_zero<CTRL, ROWS>((uint32_t)(x >> 32)) << 32) | dpp_or_zero<CTRL, ROWS>((uint32_t)x);
}
__device__ __forceinline__ uint64_t readlane64(uint64_t x, int l) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), l);
    return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v) {
    v += dpp_or_zero64<0x111, 0xF>(v);
    v += dpp_or_zero64<0x112, 0xF>(v);
    v += dpp_or_zero64<0x114, 0xF>(v);
    v += dpp_or_zero64<0x118, 0xF>(v);
    v += dpp_or_zero64<0x142, 0xA>(v);
    v += dpp_or_zero64<0x143, 0xC>(v);
    return readlane64(v, 63);
}
__device__ __forceinline__ int wave_incl_scan(int v) {
    return (int)wave_scan32((uint32_t)v, [](uint32_t a, uint32_t b) { return a + b; });
}
__device__ __forceinline__ int wave_sum_i32(int v) { return last_lane(wave_incl_scan(v)); }
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
    return (uint32_t)last_lane((int)wave_scan32(v, [](uint32_t a, uint32_t b) { return a > b ? a : b; }));
}

__device__ __forceinline__ uint32_t align2(uint32_t x) { return (x + 1u) & ~1u; }

// Global atomics are performed in L2, so a plain load issued after them may still be served
// from a stale line in this compute unit's vector L1, or overtake them.  After a phase that
// builds data with global atomics (and its barrier, if other waves read it), every reading
// wave waits for its memory operations and invalidates the L1.  While data is built it is one
// workgroup's own, hence on one compute unit and one L2: the L2 stays valid.  (A top-level list
// that other workgroups read later is released and acquired at device scope, see move_top_list
// and the helper's start in search_kernel; an arena slot that changes hands is released so too.)
// Wait until this wave's memory operations are done, so that plain stores made by some
// lanes are in place before other lanes load them.
__device__ __forceinline__ void wait_mem() { __builtin_amdgcn_s_waitcnt(0); }

// The same where only some lanes come by, and for the compiler too: what follows is read after
// what precedes has arrived.
__device__ __forceinline__ void wait_loads() {
    __builtin_amdgcn_s_waitcnt(0);
    asm volatile("" ::: "memory");
}

__device__ __forceinline__ void see_atomics() {
    __builtin_amdgcn_s_waitcnt(0);
    asm volatile("buffer_inv sc0" ::: "memory");
}

// Whether the graph of work-list entry ti has been cancelled by the host (batched calls of a
// server only): the word lives in host memory, so it is read at system scope.
__device__ __forceinline__ bool root_cancelled(const SearchArgs &a, int64_t ti) {
    if (!a.cancel || !a.tasks) return false;
    const int g = (int)(a.tasks[ti] >> 32);
    return __hip_atomic_load(a.cancel + g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) != 0u;
}

// Workgroup memory (LDS) pointers carry their address space, so that accesses and atomics
// through them are LDS instructions even where the compiler cannot trace them to the shared
// array (through a generic pointer they would be flat instructions).
typedef __attribute__((address_space(3))) uint32_t lds_u32;
typedef __attribute__((address_space(3))) unsigned long long lds_u64;
template <typename T>
__device__ __forceinline__ T *lds_at(unsigned char *base, size_t off) {
    return (T *)(base + off);
}
__device__ __forceinline__ uint32_t lds_add32(lds_u32 *p, uint32_t v) {
    return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_min32(lds_u32 *p, uint32_t v) {
    __hip_atomic_fetch_min(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_add64(lds_u64 *p, uint64_t v) {
    __hip_atomic_fetch_add(p, (unsigned long long)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_add(void *p, uint64_t v) {
    __hip_atomic_fetch_add((lds_u64 *)p, (unsigned long long)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_max(void *p, uint64_t v) {
    __hip_atomic_fetch_max((lds_u64 *)p, (unsigned long long)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_or(void *p, uint64_t v) {
    __hip_atomic_fetch_or((lds_u64 *)p, (unsigned long long)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// Set bits of a rank-bitmap word, in the workgroup's arena slot or in LDS.
__device__ __forceinline__ void bm_or(uint64_t *p, uint64_t v) {
    atomicOr(reinterpret_cast<unsigned long long *>(p), (unsigned long long)v);
}
__device__ __forceinline__ void bm_or(lds_u64 *p, uint64_t v) {
    __hip_atomic_fetch_or(p, (unsigned long long)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// ------------------------------------------------------------------------------ frames

// Registers of the frame a wave is working on; saved whole in the header array on descent.
struct FrameState {
    uint32_t off;    // 32-bit-word offset of the frame's data in the wave stack, or kShared
    uint32_t top;    // first free stack word above this frame
    int32_t n;       // list positions: [0, nq) Q entries (rows only), [nq, n) the candidates
    int32_t nq;
    int32_t level;   // search depth of the candidates taken from this list (top level = 1)
    int32_t nL;      // |L| of the nodes below
    int32_t narrow;  // 1: one-word masks of compressed positions of R, mapped by orig[] to N(x) positions
    int32_t chunk;   // base position of the current 64-candidate chunk
    int32_t rbits;   // rows held by the frame: mask bits [0, rbits) can be set
    int32_t nm;      // the method's |P| + |Q| of the list, tallies of diagnostics mode only
    uint64_t heavy;  // lanes of the current chunk still to be handled one by one
    uint64_t sL;     // sum of the L-side hash terms of L
    uint64_t fw;     // sum over the list of (2 + deg v), byte tally only
};
// (an arena slot holds one header per depth and wave: its size is part of what a caller's memory has
// room for)
static_assert(sizeof(FrameState) == 64, "frame headers");

__device__ __forceinline__ FrameState uni_frame(const FrameState &f) {
    FrameState u;
    u.off = uni(f.off);
    u.top = uni(f.top);
    u.n = uni(f.n);
    u.nq = uni(f.nq);
    u.level = uni(f.level);
    u.nL = uni(f.nL);
    u.narrow = uni(f.narrow);
    u.chunk = uni(f.chunk);
    u.rbits = uni(f.rbits);
    u.heavy = uni(f.heavy);
    u.sL = uni(f.sL);
    u.fw = uni(f.fw);
    u.nm = uni(f.nm);
    return u;
}

// Word layout of a frame's data starting at a 2-aligned offset o (np = n - nq candidates; tb table
// bits, see table_bits):
//   ids[n] | hs[np] (u64) | masks[np][wf] (u64) | H[tb] (u64) | hR[tb] (u64) | first[tb] | cnt[tb] |
//   orig[tb] | rows[rbits][nw] (u64), nw = ceil(n / 64)
// ids are universe indices; a child frame has them in diagnostics mode only.  hs is the L-side
// hash term and masks the mask of each candidate.  Row b is the position bitmap of mask bit b:
// bit k % 64 of its word k / 64 is set when entry k holds bit b; only bits [0, rbits) can be
// set (rbits = |R| for a compressed frame).  Q entries exist in the rows alone: all a Q entry
// ever does is witness that some R'' below is not maximal, which is an AND of rows, so it
// needs no mask, hash term or id of its own.
// first / cnt / H: per bit, 1 + the first candidate position holding it, or 0 when some Q entry
// holds it (a Q entry with a single bit of R witnesses nothing else: outside diagnostics mode it
// is left out of the rows); how many candidates hold it, and the sum of their hash terms
// (valid for bits below rbits).  hR and orig: narrow frames only.
struct FrameView {
    const uint32_t *ids;
    const uint64_t *hs;
    const uint64_t *masks;
    uint32_t *first;
    uint32_t *cnt;
    uint64_t *H;
    uint32_t *orig;
    uint64_t *hR;  // (narrow frames) the R-side hash term of each bit: hvl[orig[b]]
    uint64_t *rows;
    int nw;
};

// Entries of a frame's per-bit tables: a narrow frame's own bits, else whole mask words.  (A frame
// with tables for 64 bits whatever |R| had 448 words of them; most frames of sparse graphs hold
// fewer than ten bits.)
__device__ __forceinline__ uint32_t table_bits(bool narrow, int wf, int rbits) {
    return narrow ? (uint32_t)rbits : 64u * (uint32_t)wf;
}

__device__ __forceinline__ uint32_t frame_words_fixed(int n, int nq, int wf, int rbits, bool narrow, bool ids) {
    const uint32_t tb = table_bits(narrow, wf, rbits), nw = ((uint32_t)n + 63u) >> 6, np = (uint32_t)(n - nq);
    uint32_t o = ids ? align2((uint32_t)n) : 0u;
    o += 2u * np;                           // hs
    o += 2u * np * (uint32_t)wf;            // masks
    o += 4u * tb;                           // H, first, cnt
    o += narrow ? align2(3u * tb) : 0u;     // hR, orig
    o += 2u * (uint32_t)rbits * nw;         // rows
    return o;
}

__device__ __forceinline__ FrameView frame_view(uint32_t *base, int n, int nq, int wf, int rbits, bool narrow, bool ids) {
    const uint32_t tb = table_bits(narrow, wf, rbits), np = (uint32_t)(n - nq);
    FrameView v;
    v.nw = (n + 63) >> 6;
    v.ids = base;
    uint32_t o = ids ? align2((uint32_t)n) : 0u;
    v.hs = reinterpret_cast<const uint64_t *>(base + o);
    o += 2u * np;
    v.masks = reinterpret_cast<const uint64_t *>(base + o);
    o += 2u * np * (uint32_t)wf;
    v.H = reinterpret_cast<uint64_t *>(base + o);
    o += 2u * tb;
    v.hR = reinterpret_cast<uint64_t *>(base + o);
    if (narrow) o += 2u * tb;
    v.first = base + o;
    v.cnt = v.first + tb;
    v.orig = v.cnt + tb;
    o += narrow ? align2(3u * tb) : 2u * tb;
    v.rows = reinterpret_cast<uint64_t *>(base + o);
    return v;
}

// 64 x 64 bit-matrix transpose across the wave: on entry lane i holds row i (bit j is element
// (i, j)), on return lane j holds column j (bit i is element (i, j)).  Recursive block swap:
// at block size s, the upper-right and lower-left s x s blocks trade places.  Size 32 swaps
// register halves between the wave's halves, 16 and 8 move whole bytes (one byte permute each,
// its selector depending on the lane), 4, 2 and 1 shift and merge.
__device__ __forceinline__ uint64_t wave_transpose64(uint64_t x) {
    const uint32_t ln = (uint32_t)lane_id();
    auto s32 = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)(x >> 32), false, false);
    uint32_t h[2] = {(uint32_t)s32[0], (uint32_t)s32[1]};
    // byte selectors: sources 0-3 are the second operand's bytes, 4-7 the first's
    const uint32_t sel16 = (ln & 16u) ? 0x03020706u : 0x01000504u;  // odd rows keep the high halves
    const uint32_t sel8 = (ln & 8u) ? 0x07030501u : 0x02060004u;
    const bool b4 = ln & 4u, b2 = ln & 2u, b1 = ln & 1u;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        uint32_t v = h[q];
        auto s16 = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        v = __builtin_amdgcn_perm((uint32_t)s16[0], (uint32_t)s16[1], sel16);
        uint32_t y = dpp_mov<0x128>(v);  // row_ror:8, lane ^ 8
        v = __builtin_amdgcn_perm(v, y, sel8);
        y = dpp_mov<0x1B>(dpp_mov<0x141>(v));  // half mirror, then quad mirror: lane ^ 4
        v = b4 ? ((v & 0xF0F0F0F0u) | ((y >> 4) & 0x0F0F0F0Fu)) : ((v & 0x0F0F0F0Fu) | ((y << 4) & 0xF0F0F0F0u));
        y = dpp_mov<0x4E>(v);  // lane ^ 2
        v = b2 ? ((v & 0xCCCCCCCCu) | ((y >> 2) & 0x33333333u)) : ((v & 0x33333333u) | ((y << 2) & 0xCCCCCCCCu));
        y = dpp_mov<0xB1>(v);  // lane ^ 1
        v = b1 ? ((v & 0xAAAAAAAAu) | ((y >> 1) & 0x55555555u)) : ((v & 0x55555555u) | ((y << 1) & 0xAAAAAAAAu));
        h[q] = v;
    }
    return ((uint64_t)h[1] << 32) | h[0];
}

struct Ctx {
    const int32_t *gid;    // universe global ids
    const uint64_t *M;     // universe masks (records only)
    const uint64_t *hvl;   // R-side hash term per position of N(x_root)
    const uint32_t *degl;  // degree per position of N(x_root)
    const int32_t *row;    // N(x_root)
    const int32_t *c_off;
    uint32_t *s1;                     // the workgroup's top-level list frame
    uint32_t *stk;                    // this wave's stack
    uint32_t *stu;                    // a maximal node's Q' and P' positions in list order
    uint32_t *stu_l;                  // the same in this wave's LDS (lists of at most kStuLds entries)
    lds_u32 *tl_cnt;                  // this wave's LDS list of candidates to test (64)
    lds_u64 *tl_H;                    // this wave's LDS hash sums of a narrow child (64)
    lds_u64 *qk;                      // this wave's LDS list of Q' masks (kQKeep)
    lds_u64 *pm;                      // P' masks of a child list of at most 64 (the second half of stu_l)
    lds_u32 *hist;                    // this wave's LDS histogram
    int64_t scap;
    int32_t x_root, s0, c_is_v, Wroot;
    int32_t cbase, obase;  // first packed id of the current graph's candidate / other side
    // records: rows and universe indices of the top-level list, the row words, and the universe
    // entries that hold all of N(x_root) (they are in no list)
    const uint64_t *trows;
    const uint32_t *tids;
    int tnw, tfull, rec_batch;
    lds_u64 *res;  // this wave's reserve of the record arena: ints from, index from, left (ints,
                   // indices << 32), records in the next reservation of each; NULL: none is kept
    int32_t *rec;
    unsigned long long rec_cap, rec_offs_cap;
    unsigned long long *rec_offs;
    unsigned long long *acc;
    unsigned int *flags;
};

struct WaveAcc {  // per-lane partial tallies, summed over the wave at the end
    uint64_t count, hash, out_ints, nodes, nonmax, bytes;
    uint64_t dbytes;  // design-byte tally (TB instances): global bytes this search's loads and stores request
    uint32_t max_depth;
    uint64_t ph[PH_COUNT];  // cycles per phase (wave-uniform; diagnostics only)
};

// Hash terms use the graph's own ids (packed id minus the graph's base).
__device__ __forceinline__ uint64_t hl(const Ctx &c, int32_t v) {
    return c.c_is_v ? hash_v(v - c.cbase) : hash_u(v - c.cbase);
}
__device__ __forceinline__ uint64_t hr(const Ctx &c, int32_t w) {
    return c.c_is_v ? hash_u(w - c.obase) : hash_v(w - c.obase);
}

__device__ __forceinline__ uint32_t *frame_base(const Ctx &c, uint32_t off) { return off == kShared ? c.s1 : c.stk + off; }

__device__ __forceinline__ uint32_t root_pos(const FrameState &F, const FrameView &v, uint32_t b) {
    return F.narrow ? v.orig[b] : b;
}

// The R-side hash term of frame bit b: narrow frames keep it per bit (hR), other frames'
// bits are positions of N(x) already.
__device__ __forceinline__ uint64_t root_hash(const Ctx &c, const FrameState &F, const FrameView &v, uint32_t b) {
    return F.narrow ? v.hR[b] : c.hvl[b];
}
__device__ __forceinline__ uint64_t deg_of(const Ctx &c, uint32_t li) {
    const int32_t g = c.gid[li];
    return (uint64_t)(c.c_off[g + 1] - c.c_off[g]);
}

// Stable counting sort of n staged (parent position, key) pairs by key (keys in [1, nbins));
// sorted slot s receives parent position p through put(s, p).  One wave.
template <typename Put>
__device__ __forceinline__ void wave_sort_by_key(const uint32_t *src, const uint32_t *key_of, int n, int nbins, lds_u32 *hist,
                                 Put put) {
    const int ln = lane_id();
    const uint64_t below = lanes_below();
    for (int b = ln; b < nbins; b += 64) hist[b] = 0;
    __builtin_amdgcn_wave_barrier();
    for (int base = 0; base < n; base += 64) {
        const int j = base + ln;
        if (j < n) lds_add32(&hist[key_of[j]], 1u);
    }
    __builtin_amdgcn_wave_barrier();
    int carry = 0;
    for (int base = 0; base < nbins; base += 64) {
        const int b = base + ln;
        const int h = b < nbins ? (int)hist[b] : 0;
        const int incl = wave_incl_scan(h);
        if (b < nbins) hist[b] = (uint32_t)(carry + incl - h);
        carry += last_lane(incl);
    }
    __builtin_amdgcn_wave_barrier();
    const int nbits = nbins <= 1 ? 1 : 32 - __clz(nbins - 1);
    for (int base = 0; base < n; base += 64) {
        const int j = base + ln;
        const bool act = j < n;
        const uint32_t key = act ? key_of[j] : 0u;
        const uint32_t p = act ? src[j] : 0u;
        uint64_t same = __ballot(act);
        for (int bit = 0; bit < nbits; ++bit) {
            const bool on = (key >> bit) & 1u;
            const uint64_t bb = __ballot(act && on);
            same &= on ? bb : ~bb;
        }
        uint32_t start = 0;
        if (act) start = hist[key];
        __builtin_amdgcn_wave_barrier();
        if (act) {
            put(start + (uint32_t)__popcll(same & below), p);
            if ((same >> ln) == 1ull) hist[key] = start + (uint32_t)__popcll(same);
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// Place of n records in the arena: the ints start at off; the first n1 of them have the indices
// from idx on, the others those from idx2 on.
struct RecPlace {
    unsigned long long off, idx, idx2;
    int n1;
    __device__ __forceinline__ unsigned long long index(int j) const {
        return j < n1 ? idx + (unsigned long long)j : idx2 + (unsigned long long)(j - n1);
    }
};

// Whether records of len ints in all are asked for by themselves by a wave whose next reservation
// holds kRecInts ints for each of bi records: those of more than an eighth of it.  (Written without
// a product of len, which wraps from 2^29 ints on.)
__host__ __device__ constexpr bool by_itself(unsigned int len, unsigned int bi) { return len > kRecInts / 8u * bi; }
static_assert(kRecInts % 8u == 0u && !by_itself(8u, kRecBatch0) && by_itself(9u, kRecBatch0) &&
                  !by_itself(128u, kRecBatchMax) && by_itself(129u, kRecBatchMax) &&
                  by_itself((1u << 29) + 3u, kRecBatchMax) && by_itself(0xFFFFFFFFu, kRecBatchMax),
              "reservations of any length");

// Reserves n records of len ints in all (one wave).  The arena's counters are one address for the
// whole device, which takes an atomic every 8 to 16 ns: with two per record, listing a power-law
// graph of 20,000 x 10,000 vertices (516,620 records) took three times its search, 6.5 ms against
// 2.4 now.  So a wave keeps ints and indices in reserve (c.res, LDS) and asks for 4 to 64
// records' worth at a time, twice as much each time; records of more than an eighth of that are
// asked for by themselves.  Both counters share one 64-bit word (indices above bit 32).  Indices a
// wave has left at the end are marked as holding no record, ints left over are lost; the arena is
// sized for that.  The wide search, whose nodes
// cost far more, keeps no reserve; without room for them (c.rec_batch == 0) none is kept.
__device__ __forceinline__ RecPlace reserve_records(const Ctx &c, unsigned int len, int n) {
    const int ln = lane_id();
    RecPlace p;
    p.n1 = n;
    p.idx2 = 0;
    if (!c.res) {
        unsigned long long o = 0, x = 0;
        if (ln == 0) {
            if (c.rec_batch) {
                x = atomicAdd(&c.acc[ACC_REC_INTS], ((unsigned long long)n << 32) | len);
                o = x & 0xFFFFFFFFull;
                x >>= 32;
            } else {
                o = atomicAdd(&c.acc[ACC_REC_INTS], (unsigned long long)len);
                x = atomicAdd(&c.acc[ACC_RECORDS], (unsigned long long)n);
            }
        }
        p.off = readlane64(o, 0);
        p.idx = readlane64(x, 0);
        return p;
    }
    unsigned long long off = uni((uint64_t)c.res[0]), idx = uni((uint64_t)c.res[1]);
    const uint64_t st = uni((uint64_t)c.res[2]), gr = uni((uint64_t)c.res[3]);
    unsigned int left = (unsigned int)st, bi = (unsigned int)gr, bn = (unsigned int)(gr >> 32);
    int ileft = (int)(st >> 32);
    const bool more_i = len > left, direct = more_i && by_itself(len, bi), more_n = n > ileft;
    if (more_i || more_n) {
        const unsigned int ai = !more_i ? 0u : direct ? len : kRecInts * bi;
        const unsigned int an = more_n ? (unsigned int)(n - ileft) + bn - 1u : 0u;
        unsigned long long o = 0;
        if (ln == 0) o = atomicAdd(&c.acc[ACC_REC_INTS], ((unsigned long long)an << 32) | ai);
        o = readlane64(o, 0);
        if (more_i && !direct) {
            off = o & 0xFFFFFFFFull;
            left = ai;
        }
        if (more_i) bi = min(2u * bi, kRecBatchMax);
        p.off = direct ? o & 0xFFFFFFFFull : off;
        p.idx = idx;
        if (more_n) {
            p.n1 = ileft;
            p.idx2 = o >> 32;
            idx = p.idx2 + (unsigned long long)(n - ileft);
            ileft = (int)bn - 1;
            bn = min(2u * bn, kRecBatchMax);
        } else {
            idx += (unsigned long long)n;
            ileft -= n;
        }
    } else {
        p.off = off;
        p.idx = idx;
        idx += (unsigned long long)n;
        ileft -= n;
    }
    if (!direct) {
        off += len;
        left -= len;
    }
    __builtin_amdgcn_wave_barrier();
    if (ln == 0) {
        c.res[0] = off;
        c.res[1] = idx;
        c.res[2] = ((uint64_t)(uint32_t)ileft << 32) | left;
        c.res[3] = ((uint64_t)bn << 32) | bi;
    }
    __builtin_amdgcn_wave_barrier();
    return p;
}

// Reserve the record of a maximal biclique (one wave): where it goes, or NULL when the record
// arena is full.  The head is written, and L' / R' go to pl and pr.
__device__ __forceinline__ int32_t *record_at(const Ctx &c, int nL, int r, int32_t *&pl, int32_t *&pr) {
    const int ln = lane_id();
    const unsigned int len = 2u + (unsigned int)nL + (unsigned int)r;
    const RecPlace p = reserve_records(c, len, 1);
    if (p.off + len > c.rec_cap || p.index(0) >= c.rec_offs_cap) {
        if (ln == 0) atomicOr(c.flags, (unsigned int)FLAG_RECORD_OVERFLOW);
        return nullptr;
    }
    int32_t *o = c.rec + p.off;
    pl = o + 2 + (c.c_is_v ? r : 0);   // where L' goes
    pr = o + 2 + (c.c_is_v ? 0 : nL);  // where R' goes
    if (ln == 0) {
        o[0] = c.c_is_v ? r : nL;
        o[1] = c.c_is_v ? nL : r;
        c.rec_offs[p.index(0)] = p.off;
        pl[0] = c.x_root - c.cbase;
    }
    return o;
}

// One 64-word block of an L' as bits of the top-level list, a word per lane: its vertices go to
// pl[k..), which has room for nL.  Returns k past them.
__device__ __forceinline__ int write_members(const Ctx &c, uint64_t a, int wd, int32_t *pl, int k, int nL) {
    const int pc = __popcll(a);
    const int incl = wave_incl_scan(pc);
    int at = k + incl - pc;
    for (; a; a &= a - 1ull, ++at)
        if (at < nL)  // never past the reserved record
            pl[at] = c.gid[c.tids[64 * wd + __ffsll((unsigned long long)a) - 1]] - c.cbase;
    return k + last_lane(incl);
}

// The record of a maximal node of the fixed mask classes, R' given as r positions of N(x_root) in
// c.hist: L' = {x_root} u the entries of the top-level list that hold all of R', the AND of its
// rows, a word per lane, instead of a pass over the universe's masks.  Only where no universe
// entry holds all of N(x_root) (c.tfull == 0): those are in no list.
__device__ __forceinline__ void write_record_rows(const Ctx &c, int nL, int r) {
    const int ln = lane_id();
    int32_t *pl, *pr;
    if (!record_at(c, nL, r, pl, pr)) return;
    int k = 1;
    for (int base = 0; base < c.tnw; base += 64) {
        const int wd = base + ln;
        uint64_t a = wd < c.tnw ? ~0ull : 0ull;
        for (int t = 0; t < r; t += 4) {
            uint32_t b[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) b[q] = uni(c.hist[t + q < r ? t + q : t]);
            if (wd < c.tnw)
#pragma unroll
                for (int q = 0; q < 4; ++q) a &= c.trows[(size_t)b[q] * c.tnw + wd];
        }
        k = write_members(c, a, wd, pl, k, nL);
    }
    for (int t = ln; t < r; t += 64) pr[t] = c.row[c.hist[t]] - c.obase;
    __builtin_amdgcn_wave_barrier();  // the next node's bits go to c.hist
}

// The records of a chunk's maximal nodes of |R'| = 1 (lanes in own; lane l's R' is position rp of
// N(x_root), its L' has nL vertices), reserved together, or one by one where any has 2^24 vertices
// (the lengths of 64 such records need not add up in 32 bits).  c.tfull == 0 as above.
__device__ __forceinline__ void write_leaf_records(const Ctx &c, uint64_t own, uint32_t rp, int nL) {
    const int ln = lane_id();
    const bool apart = __ballot(((own >> ln) & 1ull) && nL >= 1 << 24) != 0ull;
#pragma unroll 1
    for (uint64_t rest = own; rest;) {
        const uint64_t now = apart ? rest & (0ull - rest) : rest;
        rest &= ~now;
        const bool mine = (now >> ln) & 1ull;
        const int len = mine ? 3 + nL : 0;
        const int incl = wave_incl_scan(len);
        const RecPlace p = reserve_records(c, (unsigned int)last_lane(incl), __popcll(now));
        const unsigned long long off = p.off + (unsigned long long)(unsigned int)(incl - len);
        const unsigned long long idx = p.index(__popcll(now & lanes_below()));
        const bool fits = mine && off + (unsigned long long)len <= c.rec_cap && idx < c.rec_offs_cap;
        if (mine && !fits) atomicOr(c.flags, (unsigned int)FLAG_RECORD_OVERFLOW);
        if (fits) {
            int32_t *o = c.rec + off;
            o[0] = c.c_is_v ? 1 : nL;
            o[1] = c.c_is_v ? nL : 1;
            c.rec_offs[idx] = off;
            o[2 + (c.c_is_v ? 1 : 0)] = c.x_root - c.cbase;
            o[2 + (c.c_is_v ? 0 : nL)] = c.row[rp] - c.obase;
        }
        for (uint64_t q = __ballot(fits); q; q &= q - 1ull) {
            const int l = __ffsll((unsigned long long)q) - 1;
            int32_t *pl = c.rec + readlane64(off, l) + 2 + (c.c_is_v ? 1 : 0);
            const uint64_t *row = c.trows + (size_t)(uint32_t)__builtin_amdgcn_readlane((int)rp, l) * c.tnw;
            const int n = __builtin_amdgcn_readlane(nL, l);
            int k = 1;
            for (int base = 0; base < c.tnw; base += 64) {
                const int wd = base + ln;
                k = write_members(c, wd < c.tnw ? row[wd] : 0ull, wd, pl, k, n);
            }
        }
    }
}

// Write the record of the maximal biclique (L', R') of a node.  R' is given as positions of
// N(x_root) (Rr, Wroot words).  L' = {x_root} u {universe v : M[v] contains R'}: every vertex
// adjacent to all of R'.  Sides are sorted later by the canonicaliser.
template <typename R>  // global or LDS words
__device__ __forceinline__ void write_record(const Ctx &c, const R *Rr, int nL, int r) {
    const int ln = lane_id();
    const uint64_t below = lanes_below();
    int32_t *pl, *pr;
    if (!record_at(c, nL, r, pl, pr)) return;
    int k = 1;
    for (int base = 0; base < c.s0; base += 64) {
        const int li = base + ln;
        bool in = li < c.s0;
        if (in) {
            const uint64_t *m = c.M + (size_t)li * c.Wroot;
            for (int w = 0; w < c.Wroot; ++w) in = in && ((m[w] & Rr[w]) == Rr[w]);
        }
        const uint64_t b = __ballot(in);
        const int at = k + __popcll(b & below);
        if (in && at < nL) pl[at] = c.gid[li] - c.cbase;  // never past the reserved record
        k += __popcll(b);
    }
    int q = 0;
    for (int w = 0; w < c.Wroot; ++w) {
        const bool in = (Rr[w] >> ln) & 1ull;
        const uint64_t b = __ballot(in);
        const int at = q + __popcll(b & below);
        if (in && at < r) pr[at] = c.row[w * 64 + ln] - c.obase;
        q += __popcll(b);
    }
}

// The lanes of chunk base (one-word masks) whose candidate is the first entry of the list to hold
// some bit: nothing earlier holds all of its R'.  Lane b turns bit b's first[] entry into a lane
// of the chunk, and the wave ORs them.
__device__ __forceinline__ uint64_t first_holders(const FrameState &F, const FrameView &v, int base) {
    const int ln = lane_id();
    const uint32_t at = ln < F.rbits ? v.first[ln] - 1u - (uint32_t)base : kNone;
    const auto either = [](uint32_t a, uint32_t b) { return a | b; };
    const uint32_t lo = wave_scan32(at < 32u ? 1u << at : 0u, either);
    const uint32_t hi = wave_scan32(at - 32u < 32u ? 1u << (at - 32u) : 0u, either);
    return ((uint64_t)(uint32_t)last_lane((int)hi) << 32) | (uint32_t)last_lane((int)lo);
}

// Maximality of the candidates of chunk base (lane l: position base + l, mask m) whose lanes are
// in hv, |R'| >= 2, frames of one-word masks: a candidate is not maximal when an earlier entry
// holds all of R', a bit below its position in the AND of R''s rows.  Returns the lanes that are
// not maximal.  Most are not, and one such test alone leaves a wave waiting for a few words, so
// the wave tests many at once: 2^lg lanes per candidate, one per row word up to the chunk's end
// (lists of up to 64 entries: every lane its own candidate, the rows held one per lane).  Handled
// one by one these tests took about a fifth of the power-law search and a third of the skewed
// one's.
template <bool DIAG, bool TB>
__device__ __forceinline__ uint64_t check_chunk(const Ctx &c, const FrameState &F, const FrameView &v, int base,
                                                uint64_t m, uint64_t hv, WaveAcc &acc) {
    const int ln = lane_id();
    const bool mine = (hv >> ln) & 1ull;
    const int words = min(v.nw, ((base + 63) >> 6) + 1);
    bool dead = false;
    if (words == 1) {
        const uint64_t row = ln < F.rbits ? v.rows[(size_t)ln * v.nw] : 0ull;
        uint64_t a = mine ? (1ull << ((base + ln) & 63)) - 1ull : 0ull;
        uint64_t mm = mine ? m : 0ull;
        while (__ballot(a != 0ull && mm != 0ull)) {
            const int b = mm ? __ffsll((unsigned long long)mm) - 1 : 0;
            const uint64_t x = __shfl(row, b);
            if (mm) a &= x;
            mm &= mm - 1ull;
        }
        dead = a != 0ull;
    } else {
        const int lg = words > 32 ? 6 : 32 - __clz(words - 1);
        const int group = 1 << lg, per = 64 >> lg, nh = __popcll(hv), rk = __popcll(hv & lanes_below());
        const int sub = ln & (group - 1), grp = ln >> lg;
        if (mine) c.tl_cnt[rk] = (uint32_t)ln;
        __builtin_amdgcn_wave_barrier();
        for (int done = 0; done < nh; done += per) {
            const bool on = done + grp < nh;
            const int src = on ? (int)c.tl_cnt[done + grp] : 0;
            const uint64_t ms = __shfl(m, src);
            const int i = base + src, wi = i >> 6;
            bool hit = false;
            for (int w0 = 0; w0 < words; w0 += group) {
                const int wd = w0 + sub;
                uint64_t a = on && !hit ? (wd < wi ? ~0ull : wd == wi ? (1ull << (i & 63)) - 1ull : 0ull) : 0ull;
                uint64_t mm = ms;
                while (__ballot(a != 0ull && mm != 0ull)) {
                    if (a != 0ull && mm != 0ull) {
                        const int b0 = __ffsll((unsigned long long)mm) - 1;
                        mm &= mm - 1ull;
                        const int b1 = mm ? __ffsll((unsigned long long)mm) - 1 : b0;
                        mm &= mm - 1ull;
                        const int b2 = mm ? __ffsll((unsigned long long)mm) - 1 : b0;
                        mm &= mm - 1ull;
                        a &= v.rows[(size_t)b0 * v.nw + wd] & v.rows[(size_t)b1 * v.nw + wd] &
                             v.rows[(size_t)b2 * v.nw + wd];
                    }
                }
                hit = hit || a != 0ull;
            }
            const uint64_t hb = __ballot(hit);
            if (mine && rk >= done && rk < done + per)
                dead = ((hb >> ((rk - done) << lg)) & (lg == 6 ? ~0ull : (1ull << group) - 1ull)) != 0ull;
        }
    }
    if (DIAG && dead) {
        const int i = base + ln;
        const uint64_t dx = deg_of(c, v.ids[i]);
        uint64_t rs = 0;
        for (uint64_t mm = m; mm; mm &= mm - 1ull)
            rs += 2ull + (uint64_t)c.degl[root_pos(F, v, (uint32_t)(__ffsll((unsigned long long)mm) - 1))];
        const uint64_t fw = F.fw - (2ull + dx);
        acc.nodes += 1;
        acc.nonmax += 1;
        if ((uint32_t)F.level > acc.max_depth) acc.max_depth = (uint32_t)F.level;
        acc.bytes += 4ull * ((2ull + dx) + (rs < fw ? rs : fw) + (uint64_t)(F.nm - 1) + (uint64_t)__popcll(m));
    }
    // the row words up to the candidate (lists of up to 64: every row once)
    if (TB && mine)
        acc.dbytes += words == 1 ? 0ull : 8ull * (uint64_t)__popcll(m) * (uint64_t)(((base + ln) >> 6) + 1);
    if (TB && ln == 0 && words == 1) acc.dbytes += 8ull * (uint64_t)F.rbits;
    return __ballot(dead);
}

// Candidates [base, base+64) of frame F: lanes with |R'| = 1 are settled here; returned are the
// lanes still to be handled one by one: |R'| >= 2, and for one-word masks maximal (with records
// on and vertices in no list, c.tfull, maximal candidates of |R'| = 1 too).
template <int WF, bool DIAG, bool ENUM, bool TB = false>
__device__ __forceinline__ uint64_t light_chunk(const Ctx &c, const FrameState &F, const FrameView &v, int base, WaveAcc &acc) {
    const uint64_t t0 = DIAG ? clock64() : 0ull;
    const int ln = lane_id();
    const int i = base + ln;
    const bool act = i < F.n;
    uint64_t m[WF];
    int r = 0;
#pragma unroll
    for (int w = 0; w < WF; ++w) {
        m[w] = act ? v.masks[(size_t)(i - F.nq) * WF + w] : 0ull;
        r += __popcll(m[w]);
    }
    bool own = false;  // |R'| = 1 and maximal: no earlier entry holds its bit
    // records of |R'| = 1 are written here, unless vertices outside the lists belong to them
    const bool here = !ENUM || c.tfull == 0;
    uint32_t rp = 0;
    int nL = 0;
    if (act && r == 1) {
        int b = 0;
#pragma unroll
        for (int w = 0; w < WF; ++w)
            if (m[w]) b = 64 * w + __ffsll((unsigned long long)m[w]) - 1;
        own = v.first[b] == (uint32_t)i + 1u;
        if (own && here) {
            // L' = L u {every entry with bit b}: all of them sit at positions >= i
            const uint64_t sL = F.sL + v.H[b];
            acc.count += 1;
            acc.hash += pair_hash(c.c_is_v, sL, root_hash(c, F, v, (uint32_t)b));
            nL = F.nL + (int)v.cnt[b];
            acc.out_ints += 3ull + (uint64_t)nL;
            if (ENUM) rp = root_pos(F, v, (uint32_t)b);
        }
        if (DIAG && (here || !own)) {
            acc.nodes += 1;
            if (!own) acc.nonmax += 1;
            if ((uint32_t)F.level > acc.max_depth) acc.max_depth = (uint32_t)F.level;
            const uint64_t dx = deg_of(c, v.ids[i]);
            const uint64_t rs = 2ull + (uint64_t)c.degl[root_pos(F, v, (uint32_t)b)];
            const uint64_t fw = F.fw - (2ull + dx);
            acc.bytes += 4ull * ((2ull + dx) + (rs < fw ? rs : fw) + (uint64_t)(F.nm - 1) + 1ull);
        }
        // first[b]; for a maximal node H[b], cnt[b], the R-side hash term (and orig[b])
        if (TB) acc.dbytes += 4ull + (own ? 20ull : 0ull);
    }
    if (TB && act) acc.dbytes += 8ull * WF;  // the entry's mask
    uint64_t hv = __ballot(act && r >= 2);
    if (DIAG) acc.ph[PH_LIGHT] += clock64() - t0;
    if constexpr (WF == 1) {
        const uint64_t t1 = DIAG ? clock64() : 0ull;
        if (hv) {
            const uint64_t open = hv & ~first_holders(F, v, base);
            if (TB && ln == 0) acc.dbytes += 4ull * (uint64_t)F.rbits;
            if (open) hv &= ~check_chunk<DIAG, TB>(c, F, v, base, m[0], open, acc);
        }
        if (DIAG) acc.ph[PH_CHECK] += clock64() - t1;
    }
    if (ENUM) {
        const uint64_t ob = __ballot(own);
        if (!here) hv |= ob;
        else if (ob) write_leaf_records(c, ob, rp, nL);
    }
    return hv;
}

// Adds to sup the subsets SET u {t, ..}, t >= T, of R''s r bits that some Q entry holds: q[t] is
// this lane's word of the Q positions holding bit t, a the AND of q over SET.  Supersets of a set
// nobody holds are passed over.
template <int T, uint32_t SET>
__device__ __forceinline__ void q_subsets(const uint64_t (&q)[6], int r, uint64_t a, uint64_t &sup) {
    if constexpr (T < 6) {
        if (T < r) {
            const uint64_t b = a & q[T];
            if (__ballot(b != 0ull)) {
                sup |= 1ull << (SET | (1u << T));
                q_subsets<T + 1, (SET | (1u << T))>(q, r, b, sup);
            }
            q_subsets<T + 1, SET>(q, r, a, sup);
        }
    }
}

// Calls f(wd, y) for the 64-position words wd (below and at the one holding position i, without
// the others; words < 64 only when in nzq) of a frame, where lane e of y is the mask, compressed
// to R''s r bits, of the entry at position 64 wd + e (0 from position i on); bt is the frame bit
// of R''s bit lane_id().  Row words are loaded four words at a time.  f returns whether to go on.
template <typename Fn>
__device__ __forceinline__ void each_q_word(const FrameView &v, int i, int r, uint32_t bt, uint64_t nzq, Fn f) {
    const int ln = lane_id(), wi = i >> 6;
    const uint64_t *row = v.rows + (size_t)bt * v.nw;
    int next = 0;
    auto step = [&]() {  // the next word to look at, or wi + 1
        while (next <= wi) {
            if (next >= 64) return next++;
            const uint64_t rest = nzq >> next;
            if (rest) {
                next += __ffsll((unsigned long long)rest);
                return next - 1;
            }
            next = 64;
        }
        return wi + 1;
    };
    bool go = true;
    while (go) {
        int wd[4];
        uint64_t x[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            wd[q] = step();
            x[q] = ln < r && wd[q] <= wi ? row[wd[q]] : 0ull;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (!go || wd[q] > wi) {
                go = false;
                continue;
            }
            go = f(wd[q], wave_transpose64(wd[q] == wi ? x[q] & ((1ull << (i & 63)) - 1ull) : x[q]));
        }
    }
}

// Q' of a compressed child, reduced to its inclusion-maximal masks of two or more bits.  A Q
// entry only ever serves as a witness that some later R'' (a subset of R') is not maximal, and
// an entry whose mask over R' lies inside another's witnesses nothing the other does not, so
// only one entry per maximal mask needs to stay.  The kept compressed masks go to c.qk.  Returns
// their number, or -1 when more than kQKeep are incomparable (then nothing is dropped).  Cost
// per 64 entries: one pass over the kept masks, and one over the word's candidates.
__device__ __forceinline__ int reduce_q(const Ctx &c, const FrameView &v, int i, int r, uint32_t bt, uint64_t nzq) {
    const int ln = lane_id();
    const uint64_t below = lanes_below();
    int nk = 0;
    each_q_word(v, i, r, bt, nzq, [&](int, uint64_t x) {
        bool cand = __popcll(x) >= 2;
        for (int t = 0; t < nk; ++t) {
            const uint64_t y = c.qk[t];  // same address on every lane
            if ((x & ~y) == 0ull) cand = false;
        }
        // among this word: drop x when another candidate holds more, or the same in a lower lane
        bool keep = cand;
        for (uint64_t q = __ballot(cand); q; q &= q - 1ull) {
            const int l = __ffsll((unsigned long long)q) - 1;
            const uint64_t y = readlane64(x, l);
            if (l != ln && (x & ~y) == 0ull && (x != y || l < ln)) keep = false;
        }
        const uint64_t sb = __ballot(keep);
        if (!sb) return true;
        // kept masks inside a new survivor go (compacted in place, 64 at a time: an entry
        // only moves down, past entries already read); the survivors join
        int ns = 0;
        for (int blk = 0; blk < nk; blk += 64) {
            const int t = blk + ln;
            const uint64_t y = t < nk ? c.qk[t] : 0ull;
            bool stay = t < nk;
            for (uint64_t q = sb; q; q &= q - 1ull) {
                const uint64_t xs = readlane64(x, __ffsll((unsigned long long)q) - 1);
                if ((y & ~xs) == 0ull) stay = false;
            }
            const uint64_t stb = __ballot(stay);
            __builtin_amdgcn_wave_barrier();
            if (stay) c.qk[ns + __popcll(stb & below)] = y;
            __builtin_amdgcn_wave_barrier();
            ns += __popcll(stb);
        }
        const int nn = ns + __popcll(sb);
        if (nn > kQKeep) {
            nk = -1;
            return false;
        }
        if (keep) c.qk[ns + __popcll(sb & below)] = x;
        __builtin_amdgcn_wave_barrier();
        nk = nn;
        return true;
    });
    return nk;
}

// The maximal node a child list is built for: its position, R' and what the expansion found.
template <int WF>
struct Grown {
    uint64_t m[WF];   // R', frame bits
    int i, r;
    int qn;           // Q' entries of two or more bits (diagnostics mode: all)
    int pn;           // P' entries, their positions in stu[0, pn) in list order
    uint64_t nzq;     // words (of the first 64) holding Q' entries
    bool small;       // |R'| <= 6: sup holds the subsets of R' that Q' entries hold
    uint64_t sup;
    const uint32_t *stu;
};

// R''s bits of mask word x, compressed: bit t is the t-th bit of R' (m; t0: bits in earlier words).
__device__ __forceinline__ uint64_t compress_word(uint64_t x, uint64_t m, int t0) {
    uint32_t lo = 0, hi = 0;
    for (int t = t0; m; m &= m - 1ull, ++t) {  // uniform
        const int p = __ffsll((unsigned long long)m) - 1;
        const uint32_t half = p < 32 ? (uint32_t)x : (uint32_t)(x >> 32);
        const uint32_t bit = __builtin_amdgcn_ubfe(half, (uint32_t)p & 31u, 1u);
        if (t < 32) lo |= bit << t;
        else hi |= bit << (t - 32);
    }
    return ((uint64_t)hi << 32) | lo;
}

// The child list of a maximal node with |R'| <= 64, at the top of the wave's stack: its Q' as
// position rows, then P' stably sorted by count, masks compressed to |R'| bits.  Q' entries are
// read off the frame's rows, 64 at a time through a transpose.  Sets the layout fields of C;
// false when the stack is full.  c.hist[0, r) holds the bits of R'.
template <int WF, bool DIAG, bool TB>
__device__ __forceinline__ bool build_narrow(const Ctx &c, const FrameState &F, const FrameView &v, const Grown<WF> &g,
                                             FrameState &C, WaveAcc &acc, bool tally, uint64_t &fwc) {
    const int ln = lane_id(), r = g.r, pn = g.pn;
    const uint64_t below = lanes_below();
    const uint32_t bt = ln < r ? c.hist[ln] : 0u;
    // each bit's position of N(x), R-side hash term, and whether an entry before the node holds it
    uint32_t rp = 0, f1 = 0;
    uint64_t rh = 0;
    if (ln < r) {
        rp = root_pos(F, v, bt);
        rh = root_hash(c, F, v, bt);
        f1 = v.first[bt];
    }
    // Q': with diagnostics off, reduced to its maximal masks where that pays
    int nq2 = g.qn;
    bool listed = false;  // the Q' masks are in c.qk
    if (!DIAG && g.small) {
        // a set is maximal when no set of one more bit is held; single bits are first[]'s
        const uint64_t sup = g.sup;
        const uint64_t above = ((sup >> 1) & 0x5555555555555555ull) | ((sup >> 2) & 0x3333333333333333ull) |
                               ((sup >> 4) & 0x0F0F0F0F0F0F0F0Full) | ((sup >> 8) & 0x00FF00FF00FF00FFull) |
                               ((sup >> 16) & 0x0000FFFF0000FFFFull) | ((sup >> 32) & 0x00000000FFFFFFFFull);
        const uint64_t mx = sup & ~above & ~0x0000000100010116ull;
        if ((mx >> ln) & 1ull) c.qk[__popcll(mx & below)] = (uint64_t)ln;
        __builtin_amdgcn_wave_barrier();
        nq2 = __popcll(mx);
        listed = true;
    } else if (!DIAG && (g.qn > kQReduce || 2 * r * (((g.qn + pn + 63) >> 6) - ((pn + 64) >> 6)) > pn + 4 + 7 * (64 - r))) {
        const int nk = reduce_q(c, v, g.i, r, bt, g.nzq);
        if (nk >= 0) {
            nq2 = nk;
            listed = true;
        }
    }
    const int n2 = nq2 + pn, nw2 = (n2 + 63) >> 6;
    const uint32_t off2 = F.top;
    const uint32_t top2 = align2(off2 + frame_words_fixed(n2, nq2, 1, r, true, DIAG));
    if ((int64_t)top2 > c.scap) {
        if (ln == 0) atomicOr(c.flags, (unsigned int)FLAG_STACK_OVERFLOW);
        return false;
    }
    uint32_t *cb = c.stk + off2;
    const FrameView v2 = frame_view(cb, n2, nq2, 1, r, true, DIAG);
    uint64_t *hs2 = const_cast<uint64_t *>(v2.hs);
    uint64_t *masks2 = const_cast<uint64_t *>(v2.masks);
    int c0 = 0;  // row words written so far; entries from 64 c0 on wait in c.qk
    if (!listed && g.qn > 0) {
        int held = 0;
        each_q_word(v, g.i, r, bt, g.nzq, [&](int wd, uint64_t y) {
            const bool sel = __popcll(y) >= (DIAG ? 1 : 2);
            const uint64_t sb = __ballot(sel);
            const int at = held + __popcll(sb & below);
            if (sel) {
                c.qk[at] = y;
                if (DIAG) cb[64 * c0 + at] = v.ids[64 * wd + ln];
            }
            held += __popcll(sb);
            __builtin_amdgcn_wave_barrier();
            if (held >= 64) {
                const uint64_t t = wave_transpose64(c.qk[ln]);
                if (ln < r) v2.rows[(size_t)ln * nw2 + c0] = t;
                const uint64_t z = c.qk[64 + ln];
                __builtin_amdgcn_wave_barrier();
                c.qk[ln] = z;
                __builtin_amdgcn_wave_barrier();
                held -= 64;
                ++c0;
            }
            return true;
        });
    }
    // P' entries to their slots: stably by count among the candidates
    c.tl_H[ln] = 0ull;
    __builtin_amdgcn_wave_barrier();
    const int nbits = r <= 1 ? 1 : 32 - __clz(r - 1);
    auto load_mask = [&](int k, bool act) {  // the entry's mask over R', compressed
        uint64_t out = 0;
        int t0 = 0;
#pragma unroll
        for (int w = 0; w < WF; ++w) {
            if (!g.m[w]) continue;  // uniform
            out |= compress_word(act ? v.masks[(size_t)(k - F.nq) * WF + w] : 0ull, g.m[w], t0);
            t0 += __popcll(g.m[w]);
        }
        return out;
    };
    auto place = [&](int slot, int k, uint64_t cm) {
        const uint64_t h = v.hs[k - F.nq];
        masks2[slot] = cm;
        hs2[slot] = h;
        if (DIAG) {
            const uint32_t li = v.ids[k];
            cb[nq2 + slot] = li;
            fwc += 2ull + deg_of(c, li);
        }
        for (uint64_t mm = cm; mm; mm &= mm - 1ull) lds_add64(&c.tl_H[__ffsll((unsigned long long)mm) - 1], h);
    };
    if (pn <= 64) {
        // one entry per lane: its slot is the number of entries of a smaller count, and of the
        // same count in lower lanes
        const bool act = ln < pn;
        const int k = act ? (int)g.stu[ln] : F.nq;
        const uint64_t cm = load_mask(k, act);
        const int cnt = __popcll(cm);
        uint64_t lt = 0ull, same = __ballot(act);
        for (int bit = nbits - 1; bit >= 0; --bit) {
            const bool on = (cnt >> bit) & 1;
            const uint64_t bb = __ballot(act && on);
            lt |= on ? same & ~bb : 0ull;
            same &= on ? bb : ~bb;
        }
        if (act) {
            const int slot = __popcll(lt) + __popcll(same & below);
            c.pm[slot] = cm;
            place(slot, k, cm);
        }
        __builtin_amdgcn_wave_barrier();
    } else {
        __builtin_amdgcn_wave_barrier();
        c.hist[ln] = 0u;  // (counts are below r <= 64)
        __builtin_amdgcn_wave_barrier();
        for (int base = 0; base < pn; base += 64) {
            const int j = base + ln;
            if (j < pn) {
                const int k = (int)g.stu[j];
                int cnt = 0;
#pragma unroll
                for (int w = 0; w < WF; ++w)
                    if (g.m[w]) cnt += __popcll(v.masks[(size_t)(k - F.nq) * WF + w] & g.m[w]);  // words of R' only
                lds_add32(&c.hist[cnt], 1u);
            }
        }
        __builtin_amdgcn_wave_barrier();
        {
            const int h = (int)c.hist[ln];
            const int incl = wave_incl_scan(h);
            c.hist[ln] = (uint32_t)(incl - h);
        }
        __builtin_amdgcn_wave_barrier();
        for (int base = 0; base < pn; base += 64) {
            const int j = base + ln;
            const bool act = j < pn;
            const int k = act ? (int)g.stu[j] : F.nq;
            const uint64_t cm = load_mask(k, act);
            const int cnt = __popcll(cm);
            // stable placement among equal counts: lanes with the same count, in lane order
            uint64_t same = __ballot(act);
            for (int bit = 0; bit < nbits; ++bit) {
                const bool on = (cnt >> bit) & 1;
                const uint64_t bb = __ballot(act && on);
                same &= on ? bb : ~bb;
            }
            uint32_t start = 0;
            if (act) start = c.hist[cnt];
            __builtin_amdgcn_wave_barrier();
            if (act) {
                if ((same >> ln) == 1ull) c.hist[cnt] = start + (uint32_t)__popcll(same);
                place((int)start + __popcll(same & below), k, cm);
            }
            __builtin_amdgcn_wave_barrier();
        }
        wait_mem();  // masks2 is read by other lanes below
    }
    // the rest of the rows (the Q' tail, then P'), and each bit's first candidate and count
    uint32_t first = kNone, cnt = 0;
    for (int q = c0; q < nw2; ++q) {
        const int p = 64 * q + ln;
        uint64_t x = 0ull;
        if (p < nq2) x = c.qk[p - 64 * c0];
        else if (p < n2) x = pn <= 64 ? c.pm[p - nq2] : masks2[p - nq2];
        const uint64_t t = wave_transpose64(x);
        if (ln < r) v2.rows[(size_t)ln * nw2 + q] = t;
        const int nqb = nq2 - 64 * q;  // Q' entries among this word's
        const uint64_t tp = nqb <= 0 ? t : nqb >= 64 ? 0ull : t & (~0ull << nqb);
        if (first == kNone && tp) first = (uint32_t)(64 * q + __ffsll((unsigned long long)tp));
        cnt += (uint32_t)__popcll(tp);
    }
    if (ln < r) {
        v2.first[ln] = f1 < (uint32_t)g.i + 1u ? 0u : first;
        v2.cnt[ln] = cnt;
        v2.H[ln] = c.tl_H[ln];
        v2.orig[ln] = rp;
        v2.hR[ln] = rh;
    }
    wait_mem();
    if (TB && tally && ln == 0) {
        // Q' rows read (unless the subsets gave it), each P' entry's mask words over R' and hash
        // term in, mask and hash term out; tables, orig and hR in and out; rows
        int nzw = 0;
#pragma unroll
        for (int w = 0; w < WF; ++w) nzw += g.m[w] ? 1 : 0;
        acc.dbytes += (g.small ? 0ull : 8ull * (uint64_t)r * (uint64_t)((g.i >> 6) + 1)) +
                      (uint64_t)pn * ((pn <= 64 ? 8ull : 16ull) * (uint64_t)nzw + 24ull) + 44ull * (uint64_t)r +
                      8ull * (uint64_t)r * (uint64_t)nw2;
    }
    C.off = off2;
    C.top = top2;
    C.n = n2;
    C.nq = nq2;
    C.narrow = 1;
    C.chunk = nq2 - 64;
    C.rbits = r;
    C.heavy = 0ull;
    return true;
}

// The child list of a maximal node with |R'| > 64: masks keep the frame's W words, P' follows Q' in
// the rows.  Q' is the frame's rows of R' up to the node, position for position; or, where the words
// of the positions that are not in Q' (those holding no bit of R', with diagnostics off also those
// holding one, which first[] stands for) would take more room than the Q' entries' own ids, hash
// terms and masks would, the positions of Q' alone.
template <int W, bool DIAG, bool TB>
__device__ __forceinline__ bool build_wide(const Ctx &c, const FrameState &F, const FrameView &v, const Grown<W> &g,
                                           FrameState &C, WaveAcc &acc, bool tally, uint64_t &fwc) {
    constexpr int bits = 64 * W;
    const int ln = lane_id(), r = g.r, pn = g.pn, wi = g.i >> 6;
    const uint64_t below = lanes_below();
    const bool compact =
        (int64_t)2 * bits * (((g.i + pn + 63) >> 6) - ((g.qn + pn + 63) >> 6)) + (DIAG ? g.i - g.qn : 0) >
        (DIAG ? (int64_t)g.qn * (2 * W + 2) : (int64_t)g.qn * (2 * W + 3) + pn);
    const int nq2 = compact ? g.qn : g.i, n2 = nq2 + pn, nw2 = (n2 + 63) >> 6;
    const uint32_t off2 = F.top;
    const uint32_t top2 = align2(off2 + frame_words_fixed(n2, nq2, W, bits, false, DIAG));
    if ((int64_t)top2 > c.scap) {
        if (ln == 0) atomicOr(c.flags, (unsigned int)FLAG_STACK_OVERFLOW);
        return false;
    }
    uint32_t *cb = c.stk + off2;
    const FrameView v2 = frame_view(cb, n2, nq2, W, bits, false, DIAG);
    uint64_t *hs2 = const_cast<uint64_t *>(v2.hs);
    uint64_t *masks2 = const_cast<uint64_t *>(v2.masks);
    int q2 = 0;  // Q' positions written
    for (int base = 0; compact && base <= wi; base += 64) {
        // the words' positions of Q', a word per lane; then, a bit of R' per lane, their bits of its row
        const int wd = base + ln;
        uint64_t u = 0ull, tw = 0ull;
        for (int t = 0; t < r; t += 4) {
            uint32_t b[4];
            uint64_t x[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) b[q] = uni(c.hist[t + q < r ? t + q : t]);
#pragma unroll
            for (int q = 0; q < 4; ++q) x[q] = wd <= wi ? v.rows[(size_t)b[q] * v.nw + wd] : 0ull;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (t + q < r) tw |= u & x[q];
                u |= x[q];
            }
        }
        const uint64_t keep = (DIAG ? u : tw) & (wd < wi ? ~0ull : wd == wi ? (1ull << (g.i & 63)) - 1ull : 0ull);
        const uint64_t nz = __ballot(keep != 0ull);
        const int incl = wave_incl_scan(__popcll(keep));
        if (DIAG) {
            int at = q2 + incl - __popcll(keep);
            for (uint64_t f = keep; f; f &= f - 1ull) cb[at++] = v.ids[64 * wd + __ffsll((unsigned long long)f) - 1];
        }
        for (int t0 = 0; t0 < r; t0 += 64) {
            const bool on = t0 + ln < r;
            const uint32_t b = on ? c.hist[t0 + ln] : 0u;
            const uint64_t *src = v.rows + (size_t)b * v.nw + base;
            uint64_t *dst = v2.rows + (size_t)b * nw2;
            int at = q2;
            uint64_t out = on && (at & 63) ? dst[at >> 6] : 0ull;
            for (uint64_t z = nz; z; z &= z - 1ull) {  // uniform
                const int l = __ffsll((unsigned long long)z) - 1, sh = at & 63;
                const uint64_t k = readlane64(keep, l);
                const uint64_t x = compress_word(on ? src[l] : 0ull, k, 0);
                out |= x << sh;
                at += __popcll(k);
                if (sh + __popcll(k) >= 64) {
                    if (on) dst[(at >> 6) - 1] = out;
                    out = sh ? x >> (64 - sh) : 0ull;
                }
            }
            if (on && (at & 63)) dst[at >> 6] = out;
        }
        q2 += last_lane(incl);
    }
    for (int base = 0; !compact && base < wi; base += 64) {
        const int wd = base + ln;
        for (int t = 0; t < r; t += 4) {
            uint32_t b[4];
            uint64_t x[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) b[q] = uni(c.hist[t + q < r ? t + q : t]);
            if (wd < wi) {
#pragma unroll
                for (int q = 0; q < 4; ++q) x[q] = v.rows[(size_t)b[q] * v.nw + wd];
#pragma unroll
                for (int q = 0; q < 4; ++q) v2.rows[(size_t)b[q] * nw2 + wd] = x[q];
            }
        }
    }
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const int b = 64 * w + ln;
        const bool in = (g.m[w] >> ln) & 1ull;
        v2.first[b] = in && v.first[b] < (uint32_t)g.i + 1u ? 0u : kNone;
        v2.cnt[b] = 0u;
        v2.H[b] = 0ull;
    }
    if (DIAG && !compact)
        for (int p = ln; p < nq2; p += 64) cb[p] = v.ids[p];
    wait_mem();
    __builtin_amdgcn_wave_barrier();
    for (int b = ln; b < r; b += 64) c.hist[b] = 0u;  // counts are below r
    __builtin_amdgcn_wave_barrier();
    for (int base = 0; base < pn; base += 64) {
        const int j = base + ln;
        if (j < pn) {
            const int k = (int)g.stu[j];
            int cnt = 0;
#pragma unroll
            for (int w = 0; w < W; ++w)
                if (g.m[w]) cnt += __popcll(v.masks[(size_t)(k - F.nq) * W + w] & g.m[w]);  // words of R' only
            lds_add32(&c.hist[cnt], 1u);
        }
    }
    __builtin_amdgcn_wave_barrier();
    int carry = 0;
    for (int base = 0; base < r; base += 64) {
        const int b = base + ln;
        const int h = b < r ? (int)c.hist[b] : 0;
        const int incl = wave_incl_scan(h);
        if (b < r) c.hist[b] = (uint32_t)(carry + incl - h);
        carry += last_lane(incl);
    }
    __builtin_amdgcn_wave_barrier();
    const int nbits = 32 - __clz(r - 1);
    uint64_t tbits = 0;
    for (int base = 0; base < pn; base += 64) {
        const int j = base + ln;
        const bool act = j < pn;
        const int k = act ? (int)g.stu[j] : F.nq;
        uint64_t x[W];
        int cnt = 0;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            x[w] = act && g.m[w] ? v.masks[(size_t)(k - F.nq) * W + w] & g.m[w] : 0ull;
            cnt += __popcll(x[w]);
        }
        // stable placement among equal counts: lanes with the same count, in lane order
        uint64_t same = __ballot(act);
        for (int bit = 0; bit < nbits; ++bit) {
            const bool on = (cnt >> bit) & 1;
            const uint64_t bb = __ballot(act && on);
            same &= on ? bb : ~bb;
        }
        uint32_t start = 0;
        if (act) start = c.hist[cnt];
        __builtin_amdgcn_wave_barrier();
        if (act) {
            if ((same >> ln) == 1ull) c.hist[cnt] = start + (uint32_t)__popcll(same);
            const uint32_t slot = start + (uint32_t)__popcll(same & below);
            const uint64_t h = v.hs[k - F.nq];
            hs2[slot] = h;
            if (DIAG) {
                const uint32_t li = v.ids[k];
                cb[nq2 + (int)slot] = li;
                fwc += 2ull + deg_of(c, li);
            }
#pragma unroll
            for (int w = 0; w < W; ++w) {
                masks2[(size_t)slot * W + w] = x[w];
                uint64_t y = x[w];
                while (y) {
                    const int b = 64 * w + __ffsll((unsigned long long)y) - 1;
                    y &= y - 1ull;
                    atomicMin(&v2.first[b], (uint32_t)nq2 + slot + 1u);
                    atomicAdd(&v2.cnt[b], 1u);
                    atomicAdd(reinterpret_cast<unsigned long long *>(&v2.H[b]), (unsigned long long)h);
                }
            }
            tbits += (uint64_t)cnt;
        }
        __builtin_amdgcn_wave_barrier();
    }
    see_atomics();
    // the word in which Q' ends: its last positions, then P'
    const int sh = nq2 & 63, w0 = nq2 >> 6;
#pragma unroll
    for (int w = 0; w < W; ++w) {
        if (!g.m[w]) continue;  // uniform: rows of the other words are never read
        const size_t b = (size_t)(64 * w + ln);
        uint64_t carry = 0ull;
        if (sh && ((g.m[w] >> ln) & 1ull))
            carry = compact ? v2.rows[b * nw2 + w0] : v.rows[b * v.nw + wi] & ((1ull << sh) - 1ull);
        int q = 0;
        for (; 64 * q < pn; ++q) {
            const int e = 64 * q + ln;
            const uint64_t t = wave_transpose64(e < pn ? masks2[(size_t)e * W + w] : 0ull);
            v2.rows[b * nw2 + w0 + q] = carry | (t << sh);
            carry = sh ? t >> (64 - sh) : 0ull;
        }
        if (w0 + q < nw2) v2.rows[b * nw2 + w0 + q] = carry;
    }
    wait_mem();
    if (TB && tally) {
        // Q' rows in and out; tables cleared, each P' entry's mask words over R' (for the count
        // and the placement), hash term in, both out, its bits' table atomics; its rows
        int nzw = 0;
#pragma unroll
        for (int w = 0; w < W; ++w) nzw += g.m[w] ? 1 : 0;
        acc.dbytes += 16ull * tbits;
        if (ln == 0)
            acc.dbytes += (compact ? 16ull * (uint64_t)r * (uint64_t)(wi + 1) + 8ull * (uint64_t)r * (uint64_t)w0
                                   : 16ull * (uint64_t)r * (uint64_t)wi) +
                          8ull * (uint64_t)r + 16ull * bits +
                          (uint64_t)pn * (16ull + 24ull * (uint64_t)nzw + 8ull * W) +
                          8ull * 64ull * (uint64_t)nzw * (uint64_t)(nw2 - w0);
    }
    C.off = off2;
    C.top = top2;
    C.n = n2;
    C.nq = nq2;
    C.narrow = 0;
    C.chunk = nq2 - 64;
    C.rbits = bits;
    C.heavy = 0ull;
    return true;
}

// OR (u) and AND (a), over the bits b of R' listed in c.hist[0, r), of word wd of row b; a
// is 0 when !in.  Rows are read four at a time.
__device__ __forceinline__ void fold_rows(const Ctx &c, const FrameView &v, int r, int wd, bool in, uint64_t &u,
                                          uint64_t &a) {
    u = 0ull;
    a = ~0ull;
    for (int t = 0; t < r; t += 4) {
        const uint32_t b0 = uni(c.hist[t]);
        const uint32_t b1 = uni(c.hist[t + 1 < r ? t + 1 : t]);
        const uint32_t b2 = uni(c.hist[t + 2 < r ? t + 2 : t]);
        const uint32_t b3 = uni(c.hist[t + 3 < r ? t + 3 : t]);
        if (in) {
            const uint64_t x0 = v.rows[(size_t)b0 * v.nw + wd], x1 = v.rows[(size_t)b1 * v.nw + wd];
            const uint64_t x2 = v.rows[(size_t)b2 * v.nw + wd], x3 = v.rows[(size_t)b3 * v.nw + wd];
            u |= (x0 | x1) | (x2 | x3);
            a &= (x0 & x1) & (x2 & x3);
        }
    }
    if (!in) a = 0ull;
}

// What handling a node did: nothing below it, its child frame pushed (state in C), or a child
// frame that did not fit the stack.  After a node that pushed nothing the caller reads the
// launch's flag word, so that every wave stops soon after one of them ran out of room (the host
// then repeats the launch).
enum class Node : int { kLeaf, kPushed, kFull };

__device__ __forceinline__ bool stack_ran_out(const unsigned int *flags) {
    return (uni(__hip_atomic_load(flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) & FLAG_STACK_OVERFLOW) != 0u;
}

// The candidate at position i of frame F, |R'| = r >= 1, handled by the whole wave (one-word
// masks: known to be maximal, see light_chunk).  report = false rebuilds the child frame of a
// node another wave owns: nothing is counted or recorded.
template <int WF, int W, bool DIAG, bool ENUM, bool TB = false>
__device__ __forceinline__ Node heavy_node(const Ctx &c, const FrameState &F, const FrameView &v, int i, FrameState &C,
                           WaveAcc &acc, bool report) {
    const int ln = lane_id();
    const uint64_t below = lanes_below();
    Grown<WF> g;
    int r = 0;
#pragma unroll
    for (int w = 0; w < WF; ++w) {
        g.m[w] = uni(v.masks[(size_t)(i - F.nq) * WF + w]);  // R' (uniform)
        r += __popcll(g.m[w]);
    }
    // the bits of R', ascending, in c.hist[0, r)
    {
        int t0 = 0;
#pragma unroll
        for (int w = 0; w < WF; ++w) {
            const bool on = (g.m[w] >> ln) & 1ull;
            if (on) c.hist[t0 + __popcll(g.m[w] & below)] = (uint32_t)(64 * w + ln);
            t0 += __popcll(g.m[w]);
        }
        __builtin_amdgcn_wave_barrier();
    }
    uint64_t tp = DIAG ? clock64() : 0ull;
    uint64_t dx = 0, rs = 0;
    if constexpr (WF > 1) {
        // maximality: an earlier entry holding every bit of R' ends the node -- a position below
        // i in the AND of R''s rows.  If some bit of R' first appears at i itself, nothing
        // earlier can hold R'.
        bool first_here = false;
#pragma unroll
        for (int w = 0; w < WF; ++w)
            if (((g.m[w] >> ln) & 1ull) && v.first[64 * w + ln] == (uint32_t)i + 1u) first_here = true;
        bool nonmax = false;
        if (TB && report && ln == 0) acc.dbytes += 8ull * WF + 4ull * (uint64_t)r;  // R'; first[] of its bits
        if (!__ballot(first_here)) {
            const int wl = i >> 6;  // the word holding position i
            for (int base = 0; base <= wl; base += 64) {
                const int wd = base + ln;
                uint64_t u, a;
                fold_rows(c, v, r, wd, wd <= wl, u, a);
                if (TB && report && ln == 0) acc.dbytes += 8ull * (uint64_t)r * (uint64_t)min(64, wl + 1 - base);
                if (wd == wl) a &= (1ull << (i & 63)) - 1ull;
                if (__ballot(a != 0ull)) {
                    nonmax = true;
                    break;
                }
            }
        }
        if (DIAG) {
            const uint64_t now = clock64();
            acc.ph[PH_CHECK] += now - tp;
            tp = now;
        }
        if (nonmax) {
            if (DIAG && report) {
                dx = deg_of(c, v.ids[i]);
                uint64_t t = 0;
#pragma unroll
                for (int w = 0; w < WF; ++w)
                    if ((g.m[w] >> ln) & 1ull) t += 2ull + (uint64_t)c.degl[root_pos(F, v, (uint32_t)(64 * w + ln))];
                rs = wave_sum_u64(t);
                if (ln == 0) {
                    acc.nodes += 1;
                    acc.nonmax += 1;
                    if ((uint32_t)F.level > acc.max_depth) acc.max_depth = (uint32_t)F.level;
                    const uint64_t fw = F.fw - (2ull + dx);
                    acc.bytes += 4ull * ((2ull + dx) + (rs < fw ? rs : fw) + (uint64_t)(F.nm - 1) + (uint64_t)r);
                }
            }
            return Node::kLeaf;
        }
    } else {
        if (TB && report && ln == 0) acc.dbytes += 8ull;  // R'
    }

    // maximal.  Per word of positions: the OR of R''s rows gives the entries sharing a bit with
    // R', the AND those holding all of it (after i only, the node being maximal; they join L').
    // Of the rest, P' (after i) is listed in stu in list order.  Q' (before i) is only located:
    // for |R'| <= 6 the subsets of R' that its entries hold are found by ANDs of whole row words,
    // otherwise the entries holding two or more bits of R' are counted per word.
    int ne_l = 0, qn_l = 0, nu = 0;
    uint64_t exps = 0, fwc = 0, sup = 0, nzq = 0;
    bool joins = false;
    // (the two-word class's and wider top-level lists take all of it too)
    const bool small = !DIAG && r <= 6;
    uint32_t *const stu = F.n - F.nq <= kStuLds ? c.stu_l : c.stu;
    {
        const int wi = i >> 6;
        const uint64_t bi = 1ull << (i & 63);
        for (int base = 0; base < v.nw; base += 64) {
            const int wd = base + ln;
            const bool in = wd < v.nw;
            const uint64_t before = wd < wi ? ~0ull : (wd == wi ? bi - 1ull : 0ull);
            uint64_t u = 0ull, a = in ? ~0ull : 0ull;
            if (small) {
                uint64_t x[6];
#pragma unroll
                for (int t = 0; t < 6; ++t) {
                    x[t] = 0ull;
                    if (t < r) {
                        const uint32_t b = uni(c.hist[t]);
                        if (in) x[t] = v.rows[(size_t)b * v.nw + wd];
                    }
                }
#pragma unroll
                for (int t = 0; t < 6; ++t)
                    if (t < r) {
                        u |= x[t];
                        a &= x[t];
                        x[t] &= before;
                    }
                if (base <= wi) q_subsets<0, 0u>(x, r, ~0ull, sup);
            } else {
                uint64_t tw = 0ull;
                for (int t = 0; t < r; t += 4) {
                    uint32_t b[4];
                    uint64_t x[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) b[q] = uni(c.hist[t + q < r ? t + q : t]);
#pragma unroll
                    for (int q = 0; q < 4; ++q) x[q] = in ? v.rows[(size_t)b[q] * v.nw + wd] : 0ull;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        if (t + q < r) tw |= u & x[q];
                        u |= x[q];
                        a &= x[q];
                    }
                }
                const uint64_t qs = (DIAG ? u : tw) & before;
                qn_l += __popcll(qs);
                const uint64_t qb = __ballot(qs != 0ull);
                if (base == 0) nzq = qb;
                if (DIAG)
                    for (uint64_t f = qs; f; f &= f - 1ull)
                        fwc += 2ull + deg_of(c, v.ids[64 * wd + __ffsll((unsigned long long)f) - 1]);
            }
            if (wd == wi) {
                u &= ~bi;
                a &= ~bi;
            }
            if (__ballot(a != 0ull)) {
                joins = true;
                ne_l += __popcll(a);
                for (uint64_t f = a; f; f &= f - 1ull)
                    exps += v.hs[64 * wd + __ffsll((unsigned long long)f) - 1 - F.nq];
            }
            uint64_t pm = u & ~a & ~before;
            const uint64_t pw = __ballot(pm != 0ull);
            if (__popcll(pw) <= 8) {
                // few words: one at a time, a lane per position
                for (uint64_t q = pw; q; q &= q - 1ull) {
                    const int l = __ffsll((unsigned long long)q) - 1;
                    const uint64_t y = readlane64(pm, l);
                    if ((y >> ln) & 1ull) stu[nu + __popcll(y & below)] = (uint32_t)(64 * (base + l) + ln);
                    nu += __popcll(y);
                }
            } else {
                const int pc = __popcll(pm);
                const int incl = wave_incl_scan(pc);
                int at = nu + incl - pc;
                for (; pm; pm &= pm - 1ull) stu[at++] = (uint32_t)(64 * wd + __ffsll((unsigned long long)pm) - 1);
                nu += last_lane(incl);
            }
        }
    }
    const int pn = nu;
    const int ne = joins ? wave_sum_i32(ne_l) : 0;
    const int qn = small ? 0 : wave_sum_i32(qn_l);
    wait_mem();  // stu is read by other lanes below
    if (TB && report && ln == 0) {
        // R''s rows over every word of positions, the joiners' hash terms, the listed P' entries
        // (in global scratch: written and read back), the R-side hash terms of R'
        acc.dbytes += 8ull * (uint64_t)r * (uint64_t)v.nw + 8ull * (uint64_t)ne +
                      (stu == c.stu ? 8ull : 0ull) * (uint64_t)nu + (uint64_t)r * 8ull;
    }

    // report (L', R')
    const uint64_t sL = F.sL + v.hs[i - F.nq] + (joins ? wave_sum_u64(exps) : 0ull);
    const int nL = F.nL + 1 + ne;
    if (report) {
        uint64_t sr = 0;
#pragma unroll
        for (int w = 0; w < WF; ++w)
            if ((g.m[w] >> ln) & 1ull) sr += root_hash(c, F, v, (uint32_t)(64 * w + ln));
        sr = wave_sum_u64(sr);
        if (ln == 0) {
            acc.count += 1;
            acc.hash += pair_hash(c.c_is_v, sL, sr);
            acc.out_ints += 2ull + (uint64_t)nL + (uint64_t)r;
        }
    }
    if (ENUM && report) {
        if (c.tfull == 0) {
            // the bits' positions of N(x_root) take the bits' place in c.hist meanwhile
            __builtin_amdgcn_wave_barrier();
            if (F.narrow) {
                const uint32_t bt = ln < r ? c.hist[ln] : 0u;
                if (ln < r) c.hist[ln] = v.orig[bt];
                __builtin_amdgcn_wave_barrier();
                write_record_rows(c, nL, r);
                __builtin_amdgcn_wave_barrier();
                if (ln < r) c.hist[ln] = bt;
                __builtin_amdgcn_wave_barrier();
            } else {
                write_record_rows(c, nL, r);
            }
        } else {
            // R' as positions of N(x_root), in the Q' masks' place (an array of the lane's own went to
            // registers and took a hundred others to scratch memory)
            __builtin_amdgcn_wave_barrier();
            if (ln < W) c.qk[ln] = 0ull;
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int w = 0; w < WF; ++w)
                if ((g.m[w] >> ln) & 1ull) {
                    const uint32_t rp = root_pos(F, v, (uint32_t)(64 * w + ln));
                    bm_or(&c.qk[rp >> 6], 1ull << (rp & 63));
                }
            __builtin_amdgcn_wave_barrier();
            write_record(c, c.qk, nL, r);
            __builtin_amdgcn_wave_barrier();
        }
    }
    if (DIAG && report) {
        dx = deg_of(c, v.ids[i]);
        uint64_t t = 0;
#pragma unroll
        for (int w = 0; w < WF; ++w)
            if ((g.m[w] >> ln) & 1ull) t += 2ull + (uint64_t)c.degl[root_pos(F, v, (uint32_t)(64 * w + ln))];
        rs = wave_sum_u64(t);
        if (ln == 0) {
            acc.nodes += 1;
            if ((uint32_t)F.level > acc.max_depth) acc.max_depth = (uint32_t)F.level;
            const uint64_t fw = F.fw - (2ull + dx);
            acc.bytes += 4ull * ((2ull + dx) + (rs < fw ? rs : fw) + (uint64_t)(F.nm - 1) + (uint64_t)r + (uint64_t)pn +
                                 (uint64_t)qn);
        }
    }
    if (DIAG) {
        const uint64_t now = clock64();
        acc.ph[PH_EXPAND] += now - tp;
        tp = now;
    }
    if (pn == 0) return Node::kLeaf;

    // child frame: Q' then P' stably sorted by count; masks restricted to R' and, when
    // |R'| <= 64, compressed to |R'| bits
    g.i = i;
    g.r = r;
    g.qn = qn;
    g.pn = pn;
    g.nzq = nzq;
    g.small = small;
    g.sup = sup;
    g.stu = stu;
    bool ok;
    if constexpr (WF == 1) {
        ok = build_narrow<1, DIAG, TB>(c, F, v, g, C, acc, report, fwc);
    } else {
        ok = r <= 64 ? build_narrow<WF, DIAG, TB>(c, F, v, g, C, acc, report, fwc)
                     : build_wide<WF, DIAG, TB>(c, F, v, g, C, acc, report, fwc);
    }
    if (!ok) return Node::kFull;
    C.level = F.level + 1;
    C.nL = nL;
    C.sL = sL;
    C.fw = DIAG ? wave_sum_u64(fwc) : 0ull;
    C.nm = qn + pn;
    if (DIAG) acc.ph[PH_CHILD] += clock64() - tp;
    return Node::kPushed;
}

// A wave's third-level sharing state (kept in LDS: it is needed only between chunks).
struct WaveShare {
    int cdepth;   // depth whose chunks are claimed through slot cidx (-1: none)
    int cidx;     // that slot (index into the launch's third-level slots)
    unsigned int cepoch;
    int cfirst;   // list position of chunk 0, and the number of chunks
    int climit;
    int pend;     // a chunk claimed before the list was rebuilt (-1: none)
    int hitem;    // top-level position of the node whose list is rebuilt
    int item1;    // top-level position of the node whose list is at depth 1
    int cown;     // 1: this wave published slot cidx
    int pad[3];
};
typedef __attribute__((address_space(3))) WaveShare lds_ws;

struct WGShared {
    unsigned long long task;
    int s0;
    uint32_t claim;     // next top-level item (owner, before the list moves to the steal slot)
    uint32_t moved;     // 0: items claimed in LDS; 2: moving to the steal slot; 1: moved
    int published;      // the steal slot holds this task's list
    int nonmax;
    int pcount;
    unsigned long long exps;
    unsigned long long fw1;
    unsigned long long hvsum;
    unsigned long long rs1;
    int nexp;
    int graph;  // graph whose tallies the workgroup is holding
    int mode;   // 0 done, 1 own task, 2 stolen top-level list, 3 stolen third-level list
    int victim; // workgroup whose child list a stolen task shares
    unsigned int epoch;
    int gclaim; // chunks are claimed through the global steal slot
    int sg, sk; // graph and rank of a stolen task
    int slot;   // arena slot held by this workgroup
    int scan[16];
    unsigned long long red[16];  // per-graph tally reduction
    int held;            // the workgroup counts in a.busy
    int roots_done;      // this launch's top-level candidates are all handed out
    uint32_t busyw;      // waves holding work in the current task
    uint32_t idlew;      // waves looking for a third-level list to help with
    uint32_t npub;       // third-level lists published by the workgroup's waves
    int others_done;     // (wave 0) the other launches' top-level candidates are all handed out
    int vpub;            // mode 3: the third-level slot taken, and its epoch
    unsigned int vepoch;
    int vroot;           // modes 2 and 3: the arena slot that holds the top-level list
    uint32_t t0;         // wall clock when this workgroup began to search the current list
    int H;               // top-level items, and entries of the local universe, of the current task
    int us0;
    int tg, tk;          // graph and top-level rank of the current task
    FrameState topf;     // the top-level frame of the current task
    WaveShare ws[16];
};

// What a workgroup needs of a top-level list that another one built (the rest of it is read in
// place, in the builder's arena slot).
struct TopRec {
    FrameState top;
    int32_t H, s0;
};

// Add the workgroup's tallies to a graph's accumulators and clear them.  All threads call.
template <bool DIAG, bool TB = false>
__device__ __forceinline__ void flush_acc(WaveAcc &acc, unsigned long long *gacc, WGShared *sh) {
    const int ln = lane_id();
    uint64_t v[8];
    v[0] = wave_sum_u64(acc.count);
    v[1] = wave_sum_u64(acc.hash);
    v[2] = wave_sum_u64(acc.out_ints);
    v[3] = DIAG ? wave_sum_u64(acc.nodes) : 0ull;
    v[4] = DIAG ? wave_sum_u64(acc.nonmax) : 0ull;
    v[5] = DIAG ? wave_sum_u64(acc.bytes) : 0ull;
    v[6] = DIAG ? (uint64_t)wave_max_u32(acc.max_depth) : 0ull;
    v[7] = TB ? wave_sum_u64(acc.dbytes) : 0ull;
    if (ln == 0) {
        for (int q = 0; q < 6; ++q)
            if (v[q]) lds_add(&sh->red[q], v[q]);
        if (v[6]) lds_max(&sh->red[6], v[6]);
        if (v[7]) lds_add(&sh->red[7], v[7]);
        if (DIAG)
            for (int q = 0; q < PH_COUNT; ++q)
                if (acc.ph[q]) lds_add(&sh->red[8 + q], acc.ph[q]);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const int slot[6] = {ACC_COUNT, ACC_HASH, ACC_OUT_INTS, ACC_NODES, ACC_NONMAX, ACC_BYTES};
        for (int q = 0; q < 6; ++q) {
            if (sh->red[q]) atomicAdd(&gacc[slot[q]], sh->red[q]);
            sh->red[q] = 0ull;
        }
        if (sh->red[6]) atomicMax(&gacc[ACC_MAX_DEPTH], sh->red[6]);
        sh->red[6] = 0ull;
        if (sh->red[7]) atomicAdd(&gacc[ACC_DBYTES], sh->red[7]);
        sh->red[7] = 0ull;
        for (int q = 0; q < PH_COUNT; ++q) {
            if (sh->red[8 + q]) atomicAdd(&gacc[ACC_PHASE + q], sh->red[8 + q]);
            sh->red[8 + q] = 0ull;
        }
    }
    __syncthreads();
    acc = WaveAcc{};
}

// Claim the next n items of a top-level list moved to its steal slot: the first one's index, or
// limit once the list is used up or withdrawn.  One add: hundreds of waves may claim from one
// list, and a failed claim does no harm to a counter that only this list ever uses.
__device__ __forceinline__ int claim_items(unsigned long long *word, unsigned int epoch, int limit, int n) {
    const unsigned long long old = atomicAdd(word, (unsigned long long)n);
    return (unsigned int)(old >> 32) == epoch && (unsigned int)old < (unsigned int)limit ? (int)(unsigned int)old : limit;
}

// Claim the next step items of a published list: returns the first one's index, or -1 once
// the list is used up or its owner has moved on (epoch changed).
__device__ __forceinline__ int claim_chunk(unsigned long long *word, unsigned int epoch, int limit, unsigned int step) {
    unsigned long long old = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (;;) {
        if ((unsigned int)(old >> 32) != epoch) return -1;
        const unsigned int got = (unsigned int)old;
        if ((int)got >= limit) return -1;
        const unsigned long long prev = atomicCAS(word, old, old + (unsigned long long)step);
        if (prev == old) return (int)got;
        old = prev;
    }
}

// Block-wide exclusive prefix of popcounts over nwords bitmap words into bpre; total in
// sh->s0.  All threads call it; on return every thread sees all of bpre (a thread writes a
// run of ceil(nwords / threads) entries, so callers read entries other threads wrote).
template <typename BM, typename BP>  // global or LDS words
__device__ __forceinline__ void block_popcount_prefix(const BM *bitmap, BP *bpre, int nwords, WGShared *sh) {
    const int tid = threadIdx.x, nt = blockDim.x, wid = tid >> 6, nw = nt >> 6;
    const int per = (nwords + nt - 1) / nt;
    const int b0 = tid * per;
    int local = 0;
    for (int q = 0; q < per; ++q)
        if (b0 + q < nwords) local += __popcll(bitmap[b0 + q]);
    const int incl = wave_incl_scan(local);
    if (lane_id() == 63) sh->scan[wid] = incl;
    __syncthreads();
    if (tid == 0) {
        int run = 0;
        for (int w = 0; w < nw; ++w) {
            const int t = sh->scan[w];
            sh->scan[w] = run;
            run += t;
        }
        sh->s0 = run;
    }
    __syncthreads();
    int run = sh->scan[wid] + incl - local;
    for (int q = 0; q < per; ++q) {
        if (b0 + q < nwords) {
            bpre[b0 + q] = (uint32_t)run;
            run += __popcll(bitmap[b0 + q]);
        }
    }
    wait_mem();
    __syncthreads();
}

// Moves the unclaimed rest [r, H) of the workgroup's top-level item list to its steal slot
// and marks the LDS item counter, so later claims go to the slot.  Lane 0 of the one wave that
// set the move flag from 0 to 2 calls it; the flag becomes 1 once the slot is out.
__device__ __forceinline__ void move_top_list(const SearchArgs &a, WGShared *sh, StealSlot *slot, lds_u32 *claim_l,
                                              lds_u32 *moved_l, int g, int k, int H, unsigned int epoch) {
    const uint32_t rest = lds_add32(claim_l, kMovedMark) & (kMovedMark - 1u);
    if ((int)rest < H) {
        slot->g = g;
        slot->k = k;
        slot->limit = H;
        __threadfence();
        __hip_atomic_store(&slot->word, ((unsigned long long)epoch << 32) | rest, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        atomicAdd(a.steal_live, 1u);
        sh->published = 1;
    }
    __hip_atomic_store(moved_l, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// A wave without work looks for a published third-level list with a chunk left -- the one its
// workgroup took (thief3), else one published by a wave of its workgroup -- and claims a
// chunk.  On success the claim and the list are left in the wave's share record (the list
// sits at depth 1 once rebuilt).  Returns false once no wave of the workgroup holds work, or
// a capacity ran out.  Every exit of its loop is wave-uniform.
__device__ __forceinline__ bool find_shared_list(const SearchArgs &a, WGShared *sh, lds_ws *me, lds_u32 *busyw,
                                              lds_u32 *idlew, lds_u32 *npub, int my_slot, int nw, bool thief3) {
    const int ln = lane_id();
    if (ln == 0) lds_add32(idlew, 1u);
    bool got_one = false;
    for (bool first = true;; first = false) {
        if (uni(__hip_atomic_load(a.flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) & FLAG_RERUN) break;
        // the slots are read only while the workgroup has lists out (the list it took is
        // looked at once: its owner is in another workgroup)
        if (!(thief3 && first) && uni(__hip_atomic_load(npub, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) == 0u) {
            if (uni(__hip_atomic_load(busyw, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) == 0u) break;
            __builtin_amdgcn_s_sleep(8);
            continue;
        }
        // lane 0: the list this workgroup took; lanes 1..nw: its waves' slots
        int idx = -1;
        if (ln == 0) idx = thief3 && first ? sh->vpub : -1;
        else if (ln <= nw) idx = my_slot * a.pubw + (ln - 1);
        bool ok = false;
        unsigned int e = 0;
        int lim = 0, fi = 0, it = 0;
        if (idx >= 0) {
            PubSlot *ps = &a.pub[idx];
            const unsigned long long w1 = __hip_atomic_load(&ps->word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            e = (unsigned int)(w1 >> 32);
            if (e != 0u && (ln != 0 || e == sh->vepoch)) {
                wait_loads();
                lim = __hip_atomic_load(&ps->limit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                fi = __hip_atomic_load(&ps->first, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                it = __hip_atomic_load(&ps->i1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                wait_loads();
                const unsigned long long w2 = __hip_atomic_load(&ps->word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                ok = (unsigned int)(w2 >> 32) == e && (int)(unsigned int)w2 < lim;
            }
        }
        const uint64_t okb = __ballot(ok);
        if (okb) {
            const int src = __ffsll((unsigned long long)okb) - 1;
            idx = __builtin_amdgcn_readlane(idx, src);
            e = (unsigned int)__builtin_amdgcn_readlane((int)e, src);
            lim = __builtin_amdgcn_readlane(lim, src);
            if (ln == 0) lds_add32(busyw, 1u);  // before the claim: waiting waves see work
            int got = 0;
            if (ln == 0) got = claim_chunk(&a.pub[idx].word, e, lim, 1u);
            got = __builtin_amdgcn_readlane(got, 0);
            if (got >= 0) {
                if (ln == 0) atomicAdd(&a.acc[ACC_SHARED], 1ull);
                me->cidx = idx;
                me->cepoch = e;
                me->cfirst = __builtin_amdgcn_readlane(fi, src);
                me->climit = lim;
                me->hitem = __builtin_amdgcn_readlane(it, src);
                me->pend = got;
                me->cdepth = 1;
                got_one = true;
                break;
            }
            if (ln == 0) lds_add32(busyw, ~0u);
            continue;
        }
        // nothing to take: done once no wave of the workgroup holds work
        if (uni(__hip_atomic_load(busyw, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) == 0u) break;
        __builtin_amdgcn_s_sleep(8);
    }
    if (ln == 0) lds_add32(idlew, ~0u);
    return got_one;
}

// The classes of up to eight mask words keep four waves per SIMD resident (two 8-wave
// workgroups per compute unit), diagnostics instances apart: their register budget is capped at
// 128.  That spills some state to scratch: in the production instances 0, 36, 44 and 108 bytes per
// lane (1, 2, 4 and 8 words), in the listing instances 44, 452, 112 and 548, mostly invariants of
// the workgroup's task loop, which the search below a candidate does not read.  Capped measured
// faster than 203-234 registers at two waves per SIMD: power-law step 47.8 -> 39.1 ms, skewed
// sample 1.76 -> 1.27 s.  The search waits on memory latency, and more resident waves hide it.
// (Uncapped, the diagnostics instances spill 24 to 64 bytes.)
// TB (with DIAG and ENUM off): the production search, also tallying its design bytes.
template <int W, bool DIAG, bool ENUM, bool TB = false>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(W <= 8 && !DIAG ? 4 : 2))) void search_kernel(SearchArgs a, int64_t lo, int64_t hi, unsigned int *counter) {
    extern __shared__ unsigned char lds_raw[];
    WGShared *sh = reinterpret_cast<WGShared *>(lds_raw);
    const int tid = threadIdx.x, nt = blockDim.x, wid = uni(tid >> 6), nw = nt >> 6, ln = lane_id();
    constexpr int BITS = 64 * W;
    // third-level sharing is built into the multi-word classes only: the single-word class
    // (small top-level lists, register budget capped for residency) never publishes or helps
    constexpr bool kShare3 = W >= 2;
    const bool k3 = kShare3 && a.k3;

    // take a free arena slot (the launches of all mask classes share the slots; there are as
    // many as workgroups that can be resident at once, so one is always free)
    if (threadIdx.x == 0) {
        int got = -1;
        for (int round = 0; round < 64 && got < 0; ++round)
            for (int j = 0; j < a.nslots && got < 0; ++j) {
                const int sidx = (int)((blockIdx.x + (unsigned)j) % (unsigned)a.nslots);
                if (atomicCAS(&a.slot_busy[sidx], 0u, 1u) == 0u) got = sidx;
            }
        reinterpret_cast<WGShared *>(lds_raw)->slot = got;
        if (got < 0) atomicOr(a.flags, (unsigned int)FLAG_NO_SLOT);
    }
    __syncthreads();
    const int my_slot = reinterpret_cast<WGShared *>(lds_raw)->slot;
    if (my_slot < 0) return;
    char *wg = a.arena + (size_t)my_slot * a.lay.wg_bytes;
    uint64_t *bitmap = reinterpret_cast<uint64_t *>(wg + a.lay.off_bitmap);
    uint32_t *bpre = reinterpret_cast<uint32_t *>(wg + a.lay.off_bpre);
    uint64_t *M = reinterpret_cast<uint64_t *>(wg + a.lay.off_M);
    int32_t *gid = reinterpret_cast<int32_t *>(wg + a.lay.off_gid);
    uint32_t *cnt1 = reinterpret_cast<uint32_t *>(wg + a.lay.off_cnt);
    uint64_t *hvl = reinterpret_cast<uint64_t *>(wg + a.lay.off_hv);
    uint32_t *degl = reinterpret_cast<uint32_t *>(wg + a.lay.off_deg);
    uint32_t *t1v = reinterpret_cast<uint32_t *>(wg + a.lay.off_t1v);
    uint32_t *t1c = reinterpret_cast<uint32_t *>(wg + a.lay.off_t1c);
    uint32_t *s1 = reinterpret_cast<uint32_t *>(wg + a.lay.off_S1);
    uint64_t *hb = reinterpret_cast<uint64_t *>(wg + a.lay.off_hb);
    uint32_t *hpre = reinterpret_cast<uint32_t *>(wg + a.lay.off_hpre);
    uint32_t *hpos = reinterpret_cast<uint32_t *>(wg + a.lay.off_hpos);
    char *wv = wg + a.lay.off_waves + (size_t)wid * a.lay.wave_bytes;
    FrameState *hdr = reinterpret_cast<FrameState *>(wv + a.lay.off_w_hdr);
    const uint32_t *hposr = hpos;  // the current task's top-level items

    Ctx c;
    c.res = nullptr;
    c.c_off = a.c_off;
    c.stk = reinterpret_cast<uint32_t *>(wv + a.lay.off_w_stack);
    c.stu = reinterpret_cast<uint32_t *>(wv + a.lay.off_w_u);
    c.hist = lds_at<lds_u32>(lds_raw, sizeof(WGShared) + (size_t)wid * BITS * 4);
    {
        // per wave: candidates to test (u32[64]), a narrow child's H (u64[64]), kept Q' masks, P'
        // positions, the reserve of the record arena
        const size_t tb = sizeof(WGShared) + hist_region_bytes(BITS, nw) + (size_t)wid * kWaveLds;
        c.tl_cnt = lds_at<lds_u32>(lds_raw, tb);
        c.tl_H = lds_at<lds_u64>(lds_raw, tb + 256);
        c.qk = lds_at<lds_u64>(lds_raw, tb + 768);
        c.stu_l = reinterpret_cast<uint32_t *>(lds_raw + tb + 768 + 8 * kQKeep);
        c.pm = lds_at<lds_u64>(lds_raw, tb + 768 + 8 * kQKeep + 2 * kStuLds);
        if (ENUM && a.rec_batch) {
            c.res = lds_at<lds_u64>(lds_raw, tb + 768 + 8 * kQKeep + 4 * kStuLds);
            c.res[0] = 0ull;
            c.res[1] = 0ull;
            c.res[2] = 0ull;
            c.res[3] = ((uint64_t)kRecBatch0 << 32) | kRecBatch0;
        }
    }
    // the rank bitmap and its prefix: in LDS when the launch's graphs are small enough
    const bool rl = a.dims.nwords <= kRankLdsWords;
    lds_u64 *const lbm = lds_at<lds_u64>(lds_raw, sizeof(WGShared) + hist_region_bytes(BITS, nw) + (size_t)nw * kWaveLds);
    lds_u32 *const lbp = reinterpret_cast<lds_u32 *>(lbm + (rl ? a.dims.nwords : 0));
    auto with_rank = [&](auto &&f) {
        if (rl) f(lbm, lbp);
        else f(bitmap, bpre);
    };
    if (rl)
        for (int wd = tid; wd < a.dims.nwords; wd += nt) lbm[wd] = 0ull;
    c.scap = a.dims.scap;
    c.c_is_v = 0;
    c.cbase = 0;
    c.obase = 0;
    c.Wroot = W;
    c.rec = a.rec;
    c.rec_cap = a.rec_cap;
    c.rec_offs = a.rec_offs;
    c.rec_offs_cap = a.rec_offs_cap;
    c.rec_batch = a.rec_batch;
    c.acc = a.acc;
    c.flags = a.flags;

    WaveAcc acc{};
    bool aborted = false;
    const int ucap = a.dims.ucap;
    if (tid < 16) sh->red[tid] = 0ull;
    uint64_t t_mark = DIAG ? clock64() : 0ull;  // start of the phase being timed
    // (tally instances) this workgroup's start on the wall clock and its time finding work
    const uint64_t ld_start = TB ? wall_clock64() : 0ull;
    uint64_t ld_wait = 0;
    if (tid == 0) {
        sh->graph = -1;
        sh->held = 0;
        sh->roots_done = 0;
        sh->others_done = 0;
        sh->npub = 0u;
    }
    __syncthreads();

    for (;;) {
        if (wid == 0) {
            // a fresh top-level candidate, else a share of another workgroup's top-level list,
            // else (third-level sharing) a third-level list; with third-level sharing on, a
            // workgroup that finds none waits while others of its launch are busy, once no
            // launch has top-level candidates left (before that, leaving frees the CU for
            // the other launches).  Stop once a capacity ran out (the host reruns).
            if (ln == 0) {
                if (sh->held) atomicSub(a.busy, 1u);
                sh->held = 0;
            }
            bool waited = false;
            const uint64_t ld_w0 = TB ? wall_clock64() : 0ull;
            for (;;) {
                int mode = 0;
                unsigned int t = 0;
                if (ln == 0) {
                    const unsigned int f = __hip_atomic_load(a.flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (f & FLAG_RERUN) {
                        mode = -1;
                    } else if (!sh->roots_done) {
                        for (;;) {
                            t = atomicAdd(counter, 1u);
                            if (lo + (int64_t)t >= hi) {
                                sh->roots_done = 1;
                                break;
                            }
                            if (!root_cancelled(a, lo + (int64_t)t)) {
                                mode = 1;
                                break;
                            }
                        }
                    }
                }
                mode = __builtin_amdgcn_readlane(mode, 0);
                if (mode == 1) {
                    if (ln == 0) {
                        sh->mode = 1;
                        sh->task = t;
                        sh->epoch = t + 1u;
                    }
                    break;
                }
                if (mode < 0) {
                    if (ln == 0) sh->mode = 0;
                    break;
                }
                // a published top-level list with at least two unclaimed items, else (third-level
                // sharing) a published third-level list with at least two unclaimed chunks; 64
                // slots at a time (the two slot kinds share their head fields and stride).  Looking
                // around is done with relaxed loads, each at the coherent level by itself: an
                // acquire drops the caches of the whole compute unit and part of its L2 under the
                // workgroups still at work, again and again.  What is read is checked by the
                // word, before and after, and the one acquire comes with a task.
                bool found = false;
#pragma unroll 1
                for (int kind = 0; kind < 2 && !found; ++kind) {
                    const bool on = kind == 0 ? a.steal_on != 0 : k3;
                    // (one lane's value for all: others change it meanwhile, and the lanes of this
                    // wave must not part here)
                    if (!on || uni(__hip_atomic_load(kind == 0 ? a.steal_live : a.pub_live, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT)) == 0u)
                        continue;
                    char *arr = kind == 0 ? reinterpret_cast<char *>(a.steal) : reinterpret_cast<char *>(a.pub);
                    const int total = kind == 0 ? a.nslots : a.nslots * a.pubw;
                    const int start = kind == 0 ? my_slot : my_slot * a.pubw;
                    for (int base = 1 - kind; base < total && !found; base += 64) {  // (not its own slot)
                        const int j = base + ln;
                        bool ok = false;
                        int idx = 0, sg = 0, sk = 0, rs = 0;
                        unsigned int e = 0;
                        if (j < total) {
                            idx = (start + j) % total;
                            StealSlot *sl = reinterpret_cast<StealSlot *>(arr + (size_t)idx * sizeof(StealSlot));
                            const unsigned long long w1 =
                                __hip_atomic_load(&sl->word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            e = (unsigned int)(w1 >> 32);
                            if (e != 0u) {
                                wait_loads();
                                sg = __hip_atomic_load(&sl->g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                                sk = __hip_atomic_load(&sl->k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                                const int lim = __hip_atomic_load(&sl->limit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                                rs = kind == 0 ? idx
                                               : __hip_atomic_load(&reinterpret_cast<PubSlot *>(sl)->root, __ATOMIC_RELAXED,
                                                                   __HIP_MEMORY_SCOPE_AGENT);
                                wait_loads();
                                const unsigned long long w2 =
                                    __hip_atomic_load(&sl->word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                                // the owner has not moved on, and two or more are left
                                ok = (unsigned int)(w2 >> 32) == e && (int)(unsigned int)w2 + 2 <= lim;
                            }
                        }
                        const uint64_t okb = __ballot(ok);
                        if (okb) {
                            const int src = __ffsll((unsigned long long)okb) - 1;
                            idx = __builtin_amdgcn_readlane(idx, src);
                            sg = __builtin_amdgcn_readlane(sg, src);
                            sk = __builtin_amdgcn_readlane(sk, src);
                            rs = __builtin_amdgcn_readlane(rs, src);
                            e = (unsigned int)__builtin_amdgcn_readlane((int)e, src);
                            // counted as a reader of the list's memory first; then the slot has to
                            // hold the same list still
                            int held = 0;
                            if (ln == 0) {
                                StealSlot *sl = reinterpret_cast<StealSlot *>(arr + (size_t)idx * sizeof(StealSlot));
                                atomicAdd(&a.steal[rs].readers, 1u);
                                wait_loads();
                                const unsigned long long w3 =
                                    __hip_atomic_load(&sl->word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                                held = (unsigned int)(w3 >> 32) == e;
                                if (!held) atomicSub(&a.steal[rs].readers, 1u);
                            }
                            if (!__builtin_amdgcn_readlane(held, 0)) continue;
                            if (ln == 0) {
                                sh->mode = 2 + kind;
                                sh->vroot = rs;
                                sh->victim = idx;
                                sh->vpub = idx;
                                sh->epoch = e;
                                sh->vepoch = e;
                                sh->sg = sg;
                                sh->sk = sk;
                            }
                            found = true;
                        }
                    }
                }
                if (found) break;
                int wait = 0;
                if (ln == 0 && (k3 || a.steal_on) &&
                    __hip_atomic_load(a.busy, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > 0u) {
                    wait = 1;
                    if (!sh->others_done) {
#pragma unroll
                        for (int q = 0; q < 5; ++q)
                            if (q != a.cls && (int64_t)__hip_atomic_load(&a.cls_ctr[q], __ATOMIC_RELAXED,
                                                                         __HIP_MEMORY_SCOPE_AGENT) < a.cls_n[q])
                                wait = 0;
                        if (wait) sh->others_done = 1;  // (they stay handed out)
                    }
                }
                if (!__builtin_amdgcn_readlane(wait, 0)) {
                    if (ln == 0) sh->mode = 0;
                    break;
                }
                if (ln == 0 && !waited) atomicAdd(a.hungry, 1u);
                waited = true;
                __builtin_amdgcn_s_sleep(64);
            }
            if (ln == 0) {
                if (waited) atomicSub(a.hungry, 1u);
                if (sh->mode != 0) {
                    atomicAdd(a.busy, 1u);
                    sh->held = 1;
                }
            }
            if (TB) ld_wait += wall_clock64() - ld_w0;
        }
        __syncthreads();
        if (DIAG) {
            const uint64_t now = clock64();
            acc.ph[PH_WAIT] += now - t_mark;
            t_mark = now;
        }
        const int mode = uni(sh->mode);
        if (mode == 0) break;
        const bool thief = mode >= 2;  // the top-level node belongs to another workgroup
        const bool thief3 = kShare3 && mode == 3;
        int g = 0;
        int64_t k;
        if (thief) {
            g = uni(sh->sg);
            k = uni(sh->sk);
        } else if (a.tasks) {
            const unsigned long long tk = a.tasks[lo + (int64_t)sh->task];
            g = (int)(tk >> 32);
            k = (int64_t)(tk & 0xFFFFFFFFull);
        } else {
            k = hi - 1 - (int64_t)sh->task;  // ranks are claimed from the top (largest degree) down
        }
        if (g != sh->graph) {
            // tallies belong to the graph they were found in
            if (sh->graph >= 0) flush_acc<DIAG, TB>(acc, a.graphs[sh->graph].acc, sh);
            __syncthreads();
            if (tid == 0) sh->graph = g;
            __syncthreads();
        }
        const GraphDesc gd = a.graphs[g];
        c.c_is_v = gd.c_is_v;
        c.cbase = gd.cbase;
        c.obase = gd.obase;
        const int nwords = gd.nwords;
        const int32_t x = gd.order[k];
        const int32_t rb = a.c_off[x];
        const int32_t d = a.c_off[x + 1] - rb;
        const int32_t *row = a.c_adj + rb;
        c.row = row;
        c.x_root = x;
        // the top-level list and what belongs to it: in this workgroup's arena slot, or where
        // the list's owner built it
        const int root_slot = thief ? uni(sh->vroot) : my_slot;
        {
            char *rw = a.arena + (size_t)root_slot * a.lay.wg_bytes;
            c.gid = reinterpret_cast<int32_t *>(rw + a.lay.off_gid);
            c.M = reinterpret_cast<uint64_t *>(rw + a.lay.off_M);
            c.hvl = reinterpret_cast<uint64_t *>(rw + a.lay.off_hv);
            c.degl = reinterpret_cast<uint32_t *>(rw + a.lay.off_deg);
            c.s1 = reinterpret_cast<uint32_t *>(rw + a.lay.off_S1);
            hposr = reinterpret_cast<uint32_t *>(rw + a.lay.off_hpos);
        }
        TopRec *const rec = reinterpret_cast<TopRec *>(a.arena + (size_t)root_slot * a.lay.wg_bytes + a.lay.off_top);
        if (thief) {
            // (building the list anew cost a workgroup 0.1 to 1.2 ms, about half of all the search
            // time on a graph of 784 x 653 vertices and 40,000 edges and a ninth on the power-law
            // graph of 10^6 edges: 21.0 -> 19.5 ms there, the skewed slice 68 -> 51 ms)
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            if (tid == 0) {
                sh->topf = rec->top;
                sh->H = rec->H;
                sh->us0 = rec->s0;
                sh->t0 = (uint32_t)wall_clock64();
                sh->claim = 0u;
                sh->moved = 0u;
                sh->published = 0;
                sh->gclaim = mode == 2 ? 1 : 0;
                sh->tg = g;
                sh->tk = (int)k;
                sh->busyw = thief3 ? 0u : (uint32_t)nw;
                sh->idlew = 0u;
            }
        } else {

        // -- the 2-hop walk of x, spread over the whole workgroup: walk index t belongs to the
        //    neighbour w_j with woff[j] <= t < woff[j+1] and reads entry wbase[j] + t - woff[j]
        //    of the other side's CSR (a hub neighbour no longer holds up one wave alone)
        // (wide classes keep one neighbour per wave: their registers are spent elsewhere)
        constexpr bool kFlatWalk = W <= 2;
        lds_u32 *woff = lds_at<lds_u32>(lds_raw, sizeof(WGShared));
        lds_u32 *wbase = woff + (BITS + 1);
        if (kFlatWalk && wid == 0) {
            int carry = 0;
            for (int base = 0; base < d; base += 64) {
                const int j = base + ln;
                int dw = 0;
                if (j < d) {
                    const int32_t w = row[j];
                    const int32_t e0 = a.o_off[w];
                    dw = a.o_off[w + 1] - e0;
                    wbase[j] = (uint32_t)e0;
                }
                const int incl = wave_incl_scan(dw);
                if (j < d) woff[j] = (uint32_t)(carry + incl - dw);
                carry += last_lane(incl);
            }
            if (ln == 0) woff[d] = (uint32_t)carry;
        }
        if (kFlatWalk) __syncthreads();
        const int walk = kFlatWalk ? (int)uni(woff[d]) : 0;
        auto walk_at = [&](int t, int &j) {
            int lo = 0, hi = d - 1;  // the last neighbour whose walk starts at or before t
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if ((int)woff[mid] <= t) lo = mid;
                else hi = mid - 1;
            }
            j = lo;
            return a.o_adj[wbase[lo] + (uint32_t)(t - (int)woff[lo])];
        };

        // -- reverse scan 1: mark the ranks of all 2-hop neighbours of x
        with_rank([&](auto *bm, auto *) {
            if constexpr (kFlatWalk) {
                for (int t = tid; t < walk; t += nt) {
                    int j;
                    const int32_t v = walk_at(t, j);
                    if (v != x) {
                        const int32_t rk = a.rank[v];
                        bm_or(&bm[rk >> 6], 1ull << (rk & 63));
                    }
                }
            } else {
                for (int j = wid; j < d; j += nw) {
                    const int32_t w = row[j];
                    const int32_t e0 = a.o_off[w], e1 = a.o_off[w + 1];
                    for (int p = e0 + ln; p < e1; p += 64) {
                        const int32_t v = a.o_adj[p];
                        if (v != x) {
                            const int32_t rk = a.rank[v];
                            bm_or(&bm[rk >> 6], 1ull << (rk & 63));
                        }
                    }
                }
            }
        });
        uint64_t hv_local = 0, rs_local = 0;
        for (int j = tid; j < BITS; j += nt) {
            if (j < d) {
                const int32_t w = row[j];
                const uint64_t h = hr(c, w);
                hvl[j] = h;
                hv_local += h;
                const uint32_t dw = (uint32_t)(a.o_off[w + 1] - a.o_off[w]);
                degl[j] = dw;
                rs_local += 2ull + dw;
            } else {
                hvl[j] = 0ull;
                degl[j] = 0u;
            }
        }
        if (tid == 0) {
            sh->nonmax = 0;
            sh->pcount = 0;
            sh->exps = 0;
            sh->fw1 = 0;
            sh->hvsum = 0;
            sh->rs1 = 0;
            sh->nexp = 0;
            sh->claim = 0u;
            sh->moved = 0u;
            sh->published = 0;
            sh->gclaim = 0;
        }
        __syncthreads();
        see_atomics();  // the rank bitmap was built with atomics
        hv_local = wave_sum_u64(hv_local);
        rs_local = wave_sum_u64(rs_local);
        if (ln == 0) {
            lds_add(&sh->hvsum, hv_local);
            lds_add(&sh->rs1, rs_local);
        }

        // -- universe numbering: prefix of bitmap popcounts (rank order)
        with_rank([&](auto *bm, auto *bp) { block_popcount_prefix(bm, bp, nwords, sh); });
        wait_mem();
        __syncthreads();
        const int s0 = uni(sh->s0);
        if (s0 > ucap) {
            // the universe does not fit: clear the bitmap, note the size, skip (rerun later)
            with_rank([&](auto *bm, auto *) {
                for (int wd = tid; wd < nwords; wd += nt) bm[wd] = 0ull;
            });
            if (tid == 0) {
                atomicOr(a.flags, (unsigned int)FLAG_UNIVERSE_OVERFLOW);
                atomicMax(&a.acc[ACC_NEED_UCAP], (unsigned long long)s0);
            }
            __syncthreads();
            if (DIAG) {
                const uint64_t now = clock64();
                acc.ph[PH_ROOT] += now - t_mark;
                t_mark = now;
            }
            continue;
        }
        int nq0 = 0;
        with_rank([&](auto *bm, auto *bp) {
            nq0 = (int)bp[k >> 6] + __popcll(bm[k >> 6] & ((1ull << (k & 63)) - 1ull));
            for (int wd = tid; wd < nwords; wd += nt) {
                uint64_t bits = bm[wd];
                uint32_t pos = bp[wd];
                while (bits) {
                    const int b = __ffsll((unsigned long long)bits) - 1;
                    bits &= bits - 1ull;
                    gid[pos++] = gd.order[wd * 64 + b];
                }
            }
        });
        nq0 = uni(nq0);
        c.s0 = s0;
        for (size_t q = tid; q < (size_t)s0 * W; q += nt) M[q] = 0ull;
        wait_mem();
        __syncthreads();

        // -- reverse scan 2: M[v] gets bit j for every w_j in N(x) adjacent to v
        with_rank([&](auto *bm, auto *bp) {
            if constexpr (kFlatWalk) {
                for (int t = tid; t < walk; t += nt) {
                    int j;
                    const int32_t v = walk_at(t, j);
                    if (v != x) {
                        const int32_t rk = a.rank[v];
                        const uint32_t li =
                            bp[rk >> 6] + (uint32_t)__popcll(bm[rk >> 6] & ((1ull << (rk & 63)) - 1ull));
                        atomicOr(reinterpret_cast<unsigned long long *>(&M[(size_t)li * W + (j >> 6)]), 1ull << (j & 63));
                    }
                }
            } else {
                for (int j = wid; j < d; j += nw) {
                    const int32_t w = row[j];
                    const int32_t e0 = a.o_off[w], e1 = a.o_off[w + 1];
                    for (int p = e0 + ln; p < e1; p += 64) {
                        const int32_t v = a.o_adj[p];
                        if (v != x) {
                            const int32_t rk = a.rank[v];
                            const uint32_t li =
                                bp[rk >> 6] + (uint32_t)__popcll(bm[rk >> 6] & ((1ull << (rk & 63)) - 1ull));
                            atomicOr(reinterpret_cast<unsigned long long *>(&M[(size_t)li * W + (j >> 6)]), 1ull << (j & 63));
                        }
                    }
                }
            }
        });
        __syncthreads();
        see_atomics();  // M was built with atomics

        // -- the top-level node for x: counts, maximality against earlier ranks, expansion
        with_rank([&](auto *bm, auto *) {
            for (int wd = tid; wd < nwords; wd += nt) bm[wd] = 0ull;
        });
        {
            bool nm = false;
            int pc = 0, nexp = 0;
            uint64_t ex = 0, fw = 0;
            for (int li = tid; li < s0; li += nt) {
                int cc = 0;
#pragma unroll
                for (int w = 0; w < W; ++w) cc += __popcll(M[(size_t)li * W + w]);
                cnt1[li] = (uint32_t)cc;
                const int32_t g = gid[li];
                const uint64_t dg = DIAG ? 2ull + (uint64_t)(a.c_off[g + 1] - a.c_off[g]) : 0ull;
                if (li < nq0) {
                    if (cc == d) {
                        nm = true;
                    } else {
                        fw += dg;
                    }
                } else if (cc == d) {
                    ex += hl(c, g);
                    ++nexp;
                } else {
                    ++pc;
                    fw += dg;
                }
            }
            if (__ballot(nm) && ln == 0) atomicOr(&sh->nonmax, 1);
            ex = wave_sum_u64(ex);
            fw = wave_sum_u64(fw);
            pc = wave_sum_i32(pc);
            nexp = wave_sum_i32(nexp);
            if (ln == 0) {
                atomicAdd(&sh->pcount, pc);
                atomicAdd(&sh->nexp, nexp);
                lds_add(&sh->exps, ex);
                lds_add(&sh->fw1, fw);
            }
        }
        wait_mem();
        __syncthreads();
        const bool root_nonmax = uni(sh->nonmax) != 0;
        const int P1 = uni(sh->pcount);
        if (TB && tid == 0) {
            // x's row; its neighbours' offsets (walk set-up, hash and degree terms); both reverse
            // scans (rows, ranks and mask atomics; bitmap atomics and the universe index lookups
            // unless the bitmap is in LDS); the terms per position of N(x); bitmap prefix,
            // universe ids and bitmap clear (the bitmap's part unless in LDS); universe masks
            // cleared, then read with the counts and ids
            const uint64_t dd = (uint64_t)d, wk = (uint64_t)sh->rs1 - 2ull * dd, su = (uint64_t)s0;
            acc.dbytes += 4ull * (dd + 2ull) + 16ull * dd + (rl ? 24ull : 44ull) * wk + 12ull * BITS +
                          (rl ? 0ull : 32ull * (uint64_t)nwords) + 8ull * su + 16ull * W * su + 8ull * su;
        }
        if (tid == 0) {
            const uint64_t dx = (uint64_t)d;
            if (DIAG) {
                acc.nodes += 1;
                if (acc.max_depth < 1) acc.max_depth = 1;
                const uint64_t fwtop = gd.total_fw - (2ull + dx);
                const uint64_t rs = sh->rs1;
                uint64_t b = (2ull + dx) + (rs < fwtop ? rs : fwtop) + (uint64_t)(gd.ncand - 1) + dx;
                if (root_nonmax) acc.nonmax += 1;
                else b += (uint64_t)P1 + (uint64_t)nq0;
                acc.bytes += 4ull * b;
            }
            if (!root_nonmax) {
                const uint64_t sL = hl(c, x) + sh->exps;
                const int nL = 1 + sh->nexp;
                acc.count += 1;
                acc.hash += pair_hash(c.c_is_v, sL, sh->hvsum);
                acc.out_ints += 2ull + (uint64_t)nL + (uint64_t)d;
            }
        }
        if (ENUM && !root_nonmax && wid == 0) {
            if (ln < W) c.qk[ln] = d - 64 * ln >= 64 ? ~0ull : d > 64 * ln ? (1ull << (d - 64 * ln)) - 1ull : 0ull;
            __builtin_amdgcn_wave_barrier();
            write_record(c, c.qk, 1 + sh->nexp, d);
        }
        if (root_nonmax || P1 == 0) {
            __syncthreads();
            if (DIAG) {
                const uint64_t now = clock64();
                acc.ph[PH_ROOT] += now - t_mark;
                t_mark = now;
            }
            continue;
        }
        // -- Q1 of the list: the universe entries ranked before x (all of them meet N(x)).
        //    With diagnostics off, a single-bit mask is dropped: such an entry only witnesses
        //    that R = its bit is not maximal, which the bit's first[] entry says (0 below).  The
        //    count stays nq0 in the tallies of diagnostics mode, which keep the method's full
        //    Q1.  Lists of up to 256 are kept whole: there the pass's workgroup barriers cost
        //    more than the shorter rows save (measured).
        uint32_t *ids1 = s1;
        const bool drop1 = !DIAG && nq0 > 256;
        if (drop1) {
            const int nwq = (nq0 + 63) >> 6;
            for (int q = wid; q < nwq; q += nw) {
                const int li = 64 * q + ln;
                const uint64_t kb = __ballot(li < nq0 && cnt1[li] >= 2u);
                if (ln == 0) hb[q] = kb;
            }
            wait_mem();
            __syncthreads();
            block_popcount_prefix(hb, hpre, nwq, sh);
            for (int q = tid; q < nwq; q += nt) {
                uint64_t bits = hb[q];
                uint32_t at = hpre[q];
                while (bits) {
                    const int bb = __ffsll((unsigned long long)bits) - 1;
                    bits &= bits - 1ull;
                    ids1[at++] = (uint32_t)(64 * q + bb);
                }
            }
        } else {
            for (int li = tid; li < nq0; li += nt) ids1[li] = (uint32_t)li;
            if (tid == 0) sh->s0 = nq0;
        }
        __syncthreads();
        const int nqk = uni(sh->s0);  // Q1 entries kept in the list
        const int n1 = nqk + P1;

        // -- the top-level child list as a frame: ids Q1 (earlier ranks) ++ P1 sorted by
        //    count, masks over the positions of N(x), per-bit tables
        FrameView v1 = frame_view(s1, n1, nqk, W, d, false, true);
        if (wid == 0) {
            int pn = 0;
            for (int base = nq0; base < s0; base += 64) {
                const int li = base + ln;
                const bool act = li < s0;
                const uint32_t cc = act ? cnt1[li] : 0u;
                const bool pk = act && (int)cc < d;
                const uint64_t pb = __ballot(pk);
                if (pk) {
                    const int p = pn + __popcll(pb & lanes_below());
                    t1v[p] = (uint32_t)li;
                    t1c[p] = cc;
                }
                pn += __popcll(pb);
            }
            wait_mem();
            wave_sort_by_key(t1v, t1c, pn, d, c.hist, [&](uint32_t slot, uint32_t li) { ids1[nqk + slot] = li; });
        }
        // per-bit tables accumulated in LDS (the histograms' space, idle here, 16 bytes per
        // bit), then written out
        lds_u64 *lH = lds_at<lds_u64>(lds_raw, sizeof(WGShared));
        lds_u32 *lfirst = lds_at<lds_u32>(lds_raw, sizeof(WGShared) + (size_t)BITS * 8);
        lds_u32 *lcnt = lfirst + BITS;
        __syncthreads();  // wave 0's sort is done with its histogram
        for (int b = tid; b < BITS; b += nt) {
            lfirst[b] = kNone;
            lcnt[b] = 0u;
            lH[b] = 0ull;
        }
        wait_mem();
        __syncthreads();
        uint64_t *masks1 = const_cast<uint64_t *>(v1.masks);
        uint64_t *hs1 = const_cast<uint64_t *>(v1.hs);
        for (int j = tid; j < n1; j += nt) {
            const uint32_t li = ids1[j];
            const bool cand = j >= nqk;
            const uint64_t h = cand ? hl(c, gid[li]) : 0ull;
            if (cand) hs1[j - nqk] = h;
#pragma unroll 1
            for (int w = 0; w < W; ++w) {
                uint64_t mm = M[(size_t)li * W + w];
                if (cand) masks1[(size_t)(j - nqk) * W + w] = mm;
                while (mm) {
                    const int b = 64 * w + __ffsll((unsigned long long)mm) - 1;
                    mm &= mm - 1ull;
                    lds_min32(&lfirst[b], cand ? (uint32_t)j + 1u : 0u);
                    if (cand) {
                        lds_add32(&lcnt[b], 1u);
                        lds_add64(&lH[b], h);
                    }
                }
            }
        }
        if (drop1)
            for (int li = tid; li < nq0; li += nt)
                if (cnt1[li] == 1u) {
                    int b = 0;
#pragma unroll 1
                    for (int w = 0; w < W; ++w) {
                        const uint64_t y = M[(size_t)li * W + w];
                        if (y) b = 64 * w + __ffsll((unsigned long long)y) - 1;
                    }
                    lds_min32(&lfirst[b], 0u);
                }
        __syncthreads();
        for (int b = tid; b < BITS; b += nt) {
            v1.first[b] = lfirst[b];
            v1.cnt[b] = lcnt[b];
            v1.H[b] = lH[b];
        }
        // position rows of the top-level list, one (64-entry chunk, mask word) block per wave
        const int qd = (d + 63) >> 6;  // mask words holding bits of N(x)
        for (int job = wid; job < v1.nw * qd; job += nw) {
            const int w = job / qd, q = job - w * qd;
            const int j = 64 * w + ln;
            const uint64_t t = wave_transpose64(j < n1 ? M[(size_t)ids1[j] * W + q] : 0ull);
            if (64 * q + ln < d) v1.rows[(size_t)(64 * q + ln) * v1.nw + w] = t;
        }
        wait_mem();
        __syncthreads();

        // -- top-level light pass: chunks of P1 are split over the waves; candidates with
        //    |R'| = 1 are settled here, and those to be handled one by one are flagged per chunk
        //    and listed in order in hpos.
        FrameState top;
        top.off = kShared;
        top.top = 0;
        top.n = n1;
        top.nq = nqk;
        top.level = 2;
        top.nL = 1 + sh->nexp;
        top.narrow = 0;
        top.chunk = 0;
        top.rbits = d;
        top.heavy = 0ull;
        top.sL = hl(c, x) + sh->exps;
        top.fw = uni((uint64_t)sh->fw1);
        top.nm = nq0 + P1;
        if (ENUM) {  // for the records of the top-level light pass
            c.trows = v1.rows;
            c.tids = v1.ids;
            c.tnw = v1.nw;
            c.tfull = sh->nexp;
        }
        const int nch = (P1 + 63) >> 6;
        for (int q = wid; q < nch; q += nw) {
            const uint64_t hm = light_chunk<W, DIAG, ENUM, TB>(c, top, v1, nqk + 64 * q, acc);
            if (ln == 0) hb[q] = hm;
        }
        wait_mem();
        __syncthreads();
        block_popcount_prefix(hb, hpre, nch, sh);
        for (int q = tid; q < nch; q += nt) {
            uint64_t bits = hb[q];
            uint32_t at = hpre[q];
            while (bits) {
                const int bb = __ffsll((unsigned long long)bits) - 1;
                bits &= bits - 1ull;
                hpos[at++] = (uint32_t)(nqk + 64 * q + bb);
            }
        }
        wait_mem();
        __syncthreads();
        const int H = uni(sh->s0);
        if (TB && tid == 0) {
            // the top-level list: Q1 (pruned, or copied), P1 staged and sorted, ids / hash terms /
            // masks (universe masks read), tables, rows (list masks read, rows written), chunk
            // flags, their prefix and the item list (written, read at the claims), the header
            const uint64_t n1u = (uint64_t)n1, q0 = (uint64_t)nq0;
            uint64_t b = drop1 ? 4ull * q0 + 12ull * (uint64_t)((nq0 + 63) >> 6) + 4ull * (uint64_t)nqk +
                                     (4ull * q0 + 8ull * W * (q0 - (uint64_t)nqk))
                               : 4ull * q0;
            b += 4ull * (uint64_t)(s0 - nq0) + 20ull * (uint64_t)P1;
            b += n1u * (4ull + 8ull * W) + (uint64_t)P1 * (12ull + 8ull * W) + 16ull * BITS;
            b += (4ull + 8ull) * n1u * (uint64_t)qd + 8ull * (uint64_t)d * (uint64_t)v1.nw;
            b += 24ull * (uint64_t)nch + 8ull * (uint64_t)H + sizeof(FrameState);
            acc.dbytes += b;
        }

        if (tid == 0) {
            sh->topf = top;
            sh->t0 = (uint32_t)wall_clock64();
            sh->H = H;
            sh->us0 = s0;
            sh->tg = g;
            sh->tk = (int)k;
            sh->busyw = (uint32_t)nw;
            sh->idlew = 0u;
            rec->top = top;
            rec->H = H;
            rec->s0 = s0;
        }
        }  // (own task)

        // -- share the items.  The owner's waves claim them from an LDS counter; once a
        //    workgroup of the launch is idle, the wave whose claim notices it moves the rest of
        //    the list to the global steal slot, and from then on everyone (idle workgroups read
        //    the list in place) claims there.  A thief claims there from the start.
        StealSlot *slot = mode == 2 ? &a.steal[sh->victim] : &a.steal[my_slot];
        wait_mem();
        __syncthreads();
        const FrameState top = uni_frame(sh->topf);
        const int H = uni(sh->H);
        c.s0 = uni(sh->us0);
        if (ENUM) {
            const FrameView tv = frame_view(c.s1, top.n, top.nq, W, top.rbits, false, true);
            c.trows = tv.rows;
            c.tids = tv.ids;
            c.tnw = tv.nw;
            c.tfull = top.nL - 1;  // (a helper's too: nL counts x_root and the entries in no list)
        }
        bool gclaim = uni(sh->gclaim) != 0;
        lds_u32 *claim_l = lds_at<lds_u32>(lds_raw, offsetof(WGShared, claim));
        lds_u32 *moved_l = lds_at<lds_u32>(lds_raw, offsetof(WGShared, moved));
        const unsigned int epoch = uni(sh->epoch);
        if (DIAG) {
            const uint64_t now = clock64();
            acc.ph[PH_ROOT] += now - t_mark;
            t_mark = now;
        }

        // -- second level and below.  Each wave claims one top-level item at a time, expands
        //    it and searches depth-first below it.  With third-level sharing, a wave whose
        //    second-level list (depth 1) still has two or more chunks to go publishes it in
        //    its slot once some wave or workgroup is idle, and from then on takes that list's
        //    chunks through the slot like anyone else.  A wave left without work helps: it
        //    claims a chunk of a list published by a wave of its workgroup (or of the
        //    third-level list this workgroup took), rebuilds the list from the top-level frame
        //    (the owner's own node call, reporting nothing; lists are built deterministically)
        //    and searches the chunks it claims.  Nobody waits for a helper: every chunk is
        //    searched by the wave that claimed it, and an owner claims until none is left.
        lds_u32 *busyw = lds_at<lds_u32>(lds_raw, offsetof(WGShared, busyw));
        lds_u32 *idlew = lds_at<lds_u32>(lds_raw, offsetof(WGShared, idlew));
        lds_u32 *npub = lds_at<lds_u32>(lds_raw, offsetof(WGShared, npub));
        lds_ws *me = lds_at<lds_ws>(lds_raw, offsetof(WGShared, ws) + (size_t)wid * sizeof(WaveShare));
        me->cdepth = -1;
        me->cown = 0;
        me->hitem = -1;
        me->pend = -1;
        hdr[0] = top;  // every lane stores the same header
        wait_mem();
        bool src_top = !thief3;  // the current source: top-level items (else one published list)
        // idle workgroups of this launch, as read at the previous check (the load is issued
        // one check ahead, so its latency hides under the chunk in between)
        uint32_t hungry_seen = 0u, flags_seen = 0u;
        int inext = 0, iend = 0;  // top-level items claimed and not yet begun
        uint32_t tclaim = 0u;     // (lane 0) when, and how many, it last claimed from a moved list
        int sclaim = 1;
        for (;;) {
            if (!src_top && !find_shared_list(a, sh, me, busyw, idlew, npub, my_slot, nw, thief3)) break;
            FrameState cur = uni_frame(sh->topf);
            int depth = 0;
            while (!aborted) {
                const FrameView v = frame_view(frame_base(c, cur.off), cur.n, cur.nq, cur.narrow ? 1 : W, cur.rbits, cur.narrow != 0,
                                               DIAG || cur.off == kShared);
                int i;
                if (depth == 0) {
                    if (src_top) {
                        // a capacity that ran out elsewhere, as read at the previous claim
                        if (uni(flags_seen) & FLAG_RERUN) {
                            aborted = true;
                            break;
                        }
                        flags_seen = __hip_atomic_load(a.flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        const bool want = uni(hungry_seen) > 0u;
                        hungry_seen = __hip_atomic_load(a.hungry, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        int got = 0, mv = 0, step = 1;
                        if (inext < iend) {
                            got = inext;
                            step = iend - inext;
                        } else if (ln == 0) {
                            if (gclaim) {
                                // the counter is one address for every wave of the device: short
                                // items (by the time the last ones took) are claimed four or eight
                                // at once while many are left, long ones one by one
                                const uint32_t now = (uint32_t)wall_clock64();
                                const uint32_t per = iend > 0 ? (now - tclaim) / (uint32_t)sclaim : kLongItem;
                                step = per >= kLongItem ? 1 : max(1, min(per >= kLongItem / 4 ? 4 : 8, (H - iend) >> 6));
                                got = claim_items(&slot->word, epoch, H, step);
                                tclaim = now;
                                sclaim = step;
                            } else {
                                const uint32_t t = lds_add32(claim_l, 1u);
                                got = (int)(t & (kMovedMark - 1u));
                                if (t >= kMovedMark) {
                                    // the rest of the list went to the steal slot: wait until it
                                    // is out (the moving wave is a few stores from done), claim there
                                    while (__hip_atomic_load(moved_l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != 1u)
                                        __builtin_amdgcn_s_sleep(1);
                                    got = claim_items(&slot->word, epoch, H, 1);
                                    mv = 1;
                                } else if (uint32_t none = 0u;
                                           a.steal_on && want && got + 2 < H &&
                                           (uint32_t)wall_clock64() - sh->t0 > kShareAfter &&
                                           __hip_atomic_compare_exchange_strong(moved_l, &none, 2u, __ATOMIC_RELAXED,
                                                                               __ATOMIC_RELAXED,
                                                                               __HIP_MEMORY_SCOPE_WORKGROUP)) {
                                    // a workgroup is idle: move the rest of the list to the steal
                                    // slot (this claim keeps item got)
                                    move_top_list(a, sh, slot, claim_l, moved_l, g, (int)k, H, epoch);
                                    mv = 1;
                                }
                            }
                        }
                        got = __builtin_amdgcn_readlane(got, 0);
                        if (__builtin_amdgcn_readlane(mv, 0)) gclaim = true;
                        if (got < 0 || got >= H) break;
                        inext = got + 1;
                        iend = min(H, got + __builtin_amdgcn_readlane(step, 0));
                        i = (int)uni(hposr[got]);
                        if (k3) me->item1 = i;
                    } else {
                        // a helped list: rebuild it once (the node call below reports nothing)
                        i = uni(me->hitem);
                        if (i < 0) break;
                        me->hitem = -1;
                    }
                } else {
                    if (cur.heavy == 0ull) {
                        int base = cur.chunk + 64;
                        if (kShare3 && a.steal_on && depth == 1) {
                            if (k3 && uni(me->cdepth) == 1) {
                                int got = uni(me->pend);
                                me->pend = -1;
                                if (got < 0) {
                                    if (ln == 0) {
                                        got = claim_chunk(&a.pub[me->cidx].word, me->cepoch, me->climit, 1u);
                                        if (got >= 0 && !me->cown) atomicAdd(&a.acc[ACC_SHARED], 1ull);
                                    }
                                    got = __builtin_amdgcn_readlane(got, 0);
                                }
                                if (got >= 0) {
                                    base = uni(me->cfirst) + 64 * got;
                                } else {
                                    // every chunk is claimed: the owner withdraws the list
                                    base = cur.n;
                                    if (ln == 0 && me->cown) {
                                        __hip_atomic_store(&a.pub[me->cidx].word, 0ull, __ATOMIC_RELAXED,
                                                           __HIP_MEMORY_SCOPE_AGENT);
                                        atomicSub(a.pub_live, 1u);
                                        lds_add32(npub, ~0u);
                                    }
                                    me->cown = 0;
                                    me->cdepth = -1;
                                }
                            } else if (src_top) {
                                // idle workgroups of this launch, as read at the previous check
                                // (the load is issued one check ahead: its latency hides under
                                // the chunk in between)
                                const bool want = uni(hungry_seen) > 0u;
                                hungry_seen = __hip_atomic_load(a.hungry, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                                if (want && (uint32_t)wall_clock64() - uni(sh->t0) > kShareAfter) {
                                    // the top-level list goes out first (its items are the coarser
                                    // work): the owner's next top-level claim may be far off when
                                    // second-level subtrees are large
                                    // (the owning workgroup's list only: a thief's slot is its victim's)
                                    if (ln == 0 && mode == 1 &&
                                        __hip_atomic_load(moved_l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) == 0u &&
                                        (int)(__hip_atomic_load(claim_l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) &
                                              (kMovedMark - 1u)) + 1 < H) {
                                        uint32_t none = 0u;
                                        if (__hip_atomic_compare_exchange_strong(moved_l, &none, 2u, __ATOMIC_RELAXED,
                                                                                 __ATOMIC_RELAXED,
                                                                                 __HIP_MEMORY_SCOPE_WORKGROUP))
                                            move_top_list(a, sh, slot, claim_l, moved_l, g, (int)k, H, epoch);
                                    }
                                    if (k3 && cur.n - base > 64) {
                                        // publish the rest of this list, then claim its chunks like a helper
                                        const int idx = my_slot * a.pubw + wid;
                                        const int lim = (cur.n - base + 63) >> 6;
                                        if (ln == 0) {
                                            PubSlot *mp = &a.pub[idx];
                                            const unsigned int e = atomicAdd(a.epoch_ctr, 1u) + 1u;
                                            mp->g = sh->tg;
                                            mp->k = sh->tk;
                                            mp->i1 = me->item1;
                                            mp->first = base;
                                            mp->limit = lim;
                                            mp->root = root_slot;
                                            __threadfence();
                                            __hip_atomic_store(&mp->word, (unsigned long long)e << 32, __ATOMIC_RELAXED,
                                                               __HIP_MEMORY_SCOPE_AGENT);
                                            atomicAdd(a.pub_live, 1u);
                                            lds_add32(npub, 1u);
                                            me->cepoch = e;
                                        }
                                        me->cidx = idx;
                                        me->cfirst = base;
                                        me->climit = lim;
                                        me->cdepth = 1;
                                        me->cown = 1;
                                        continue;
                                    }
                                }
                            }
                        }
                        if (base >= cur.n) {
                            --depth;
                            cur = uni_frame(hdr[depth]);  // hdr[0] holds the top-level list
                            continue;
                        }
                        cur.chunk = base;
                        cur.heavy = (W == 1 || cur.narrow) ? light_chunk<1, DIAG, ENUM, TB>(c, cur, v, base, acc)
                                                  : light_chunk<W, DIAG, ENUM, TB>(c, cur, v, base, acc);
                        continue;
                    }
                    const int lane = __ffsll((unsigned long long)cur.heavy) - 1;
                    cur.heavy &= cur.heavy - 1ull;
                    i = cur.chunk + lane;
                }
                FrameState ch;
                const bool report = src_top || depth > 0;
                const Node node = (W == 1 || cur.narrow) ? heavy_node<1, W, DIAG, ENUM, TB>(c, cur, v, i, ch, acc, report)
                                                : heavy_node<W, W, DIAG, ENUM, TB>(c, cur, v, i, ch, acc, report);
                if (node == Node::kPushed) {
                    if (depth >= a.dims.maxdepth) {
                        if (ln == 0) atomicOr(a.flags, (unsigned int)FLAG_DEPTH_OVERFLOW);
                        aborted = true;
                        break;
                    }
                    if (depth > 0) {
                        hdr[depth] = cur;  // every lane stores the same header
                        wait_mem();
                        if (TB && ln == 0) acc.dbytes += 2ull * sizeof(FrameState);  // saved, read back on return
                    }
                    ++depth;
                    cur = ch;
                } else if (node == Node::kFull || stack_ran_out(a.flags)) {
                    aborted = true;
                }
            }
            if (!k3) break;
            // a helped list whose rebuild pushed no frame (the owner's call did; never reached)
            if (!src_top && !aborted && uni(me->pend) >= 0 && ln == 0)
                atomicOr(a.flags, (unsigned int)FLAG_SHARE_MISMATCH);
            // (after an abort) a list still published is withdrawn
            if (ln == 0 && me->cown) {
                __hip_atomic_store(&a.pub[me->cidx].word, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                atomicSub(a.pub_live, 1u);
                lds_add32(npub, ~0u);
            }
            me->cown = 0;
            me->cdepth = -1;
            me->pend = -1;
            me->hitem = -1;
            if (ln == 0) lds_add32(busyw, ~0u);  // this wave's work in the source is done
            if (aborted) break;
            src_top = false;
        }
        if (DIAG) t_mark = clock64();  // from here to the next task: waiting
        __syncthreads();
        // every chunk is claimed: withdraw the list (thieves still finish the chunks they hold)
        if (tid == 0 && sh->published) {
            atomicExch(&slot->word, 0ull);
            atomicSub(a.steal_live, 1u);
        }
        if (tid == 0 && thief) {
            wait_loads();
            atomicSub(&a.steal[root_slot].readers, 1u);
        }
    }

    if (ENUM && c.res) {  // the indices this wave has left hold no record
        const unsigned long long idx = c.res[1];
        const int ileft = (int)((uint64_t)c.res[2] >> 32);
        if (ln < ileft && idx + (unsigned long long)ln < c.rec_offs_cap) c.rec_offs[idx + (unsigned long long)ln] = kNoRecord;
    }
    // tallies of the last graph
    if (sh->graph >= 0) flush_acc<DIAG, TB>(acc, a.graphs[sh->graph].acc, sh);
    wait_mem();  // (every wave's stores to the slot have arrived before it is handed on)
    __syncthreads();
    if (threadIdx.x == 0) {
        if (TB && a.wg_load) {
            a.wg_load[3 * (size_t)blockIdx.x] = ld_start;
            a.wg_load[3 * (size_t)blockIdx.x + 1] = wall_clock64();
            a.wg_load[3 * (size_t)blockIdx.x + 2] = ld_wait;
        }
        // the arena slot goes back when no workgroup reads this one's last list any more (each
        // searches what it claimed and leaves; none waits for this one)
        while (__hip_atomic_load(&a.steal[my_slot].readers, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u)
            __builtin_amdgcn_s_sleep(32);
        __threadfence();
        atomicExch(&a.slot_busy[my_slot], 0u);
    }
}

// ============================================================================ wide roots
//
// Top-level candidates of degree above the widest mask class (64 * 16 bits) are searched by
// wide_kernel: the same method, candidate order, tree and tallies as search_kernel, in a
// simpler form whose sets may be of any width.
//  * Every frame, the top-level list included, maps its mask bits to positions of N(x)
//    through orig[], and masks below the top level are compressed to |R| bits (ceil(|R|/64)
//    words per entry), so the width shrinks with depth.
//  * A node's R' words, the list of its bits and a child's counting-sort histogram live in
//    per-wave global scratch; Q lists are kept whole.
//  * Several workgroups (replicas) rebuild the same top-level list (deterministically) and
//    claim its 64-candidate chunks from a per-candidate counter; replica 0 reports the
//    top-level node itself.

// ids[n] | hs[n] (u64) | masks[n][wf] (u64) | first[rb] | cnt[rb] | H[rb] (u64) | orig[rb] |
// rows[rb][nw] (u64) | skip[2], with wf = ceil(rb / 64), nw = ceil(n / 64); 32-bit words.
// skip[0] (pivot rule only): the number of covered candidates right after the pivot.
__device__ __forceinline__ uint64_t wframe_words(int n, int rb) {
    const uint64_t wf = ((uint64_t)rb + 63u) >> 6, nw = ((uint64_t)n + 63u) >> 6;
    uint64_t o = align2((uint32_t)n);
    o += 2ull * (uint64_t)n;
    o += 2ull * (uint64_t)n * wf;
    o += 4ull * (uint64_t)rb;  // first, cnt, H
    o += (uint64_t)rb;         // orig
    o = (o + 1ull) & ~1ull;
    o += 2ull * (uint64_t)rb * nw;
    o += 2ull;                 // skip
    return o;
}

struct WFrameView {
    const uint32_t *ids;
    const uint64_t *hs;
    const uint64_t *masks;
    uint32_t *first;
    uint32_t *cnt;
    uint64_t *H;
    uint32_t *orig;
    uint64_t *rows;
    uint32_t *skip;
    int nw, wf;
};

__device__ __forceinline__ WFrameView wframe_view(uint32_t *base, int n, int rb) {
    WFrameView v;
    v.wf = (rb + 63) >> 6;
    v.nw = (n + 63) >> 6;
    uint64_t o = align2((uint32_t)n);
    v.ids = base;
    v.hs = reinterpret_cast<const uint64_t *>(base + o);
    o += 2ull * (uint64_t)n;
    v.masks = reinterpret_cast<const uint64_t *>(base + o);
    o += 2ull * (uint64_t)n * (uint64_t)v.wf;
    v.first = base + o;
    o += (uint64_t)rb;
    v.cnt = base + o;
    o += (uint64_t)rb;
    v.H = reinterpret_cast<uint64_t *>(base + o);
    o += 2ull * (uint64_t)rb;
    v.orig = base + o;
    o += (uint64_t)rb;
    o = (o + 1ull) & ~1ull;
    v.rows = reinterpret_cast<uint64_t *>(base + o);
    o += 2ull * (uint64_t)rb * (uint64_t)v.nw;
    v.skip = base + o;
    return v;
}

// The wave's scratch of the wide search.
struct WCtx {
    Ctx c;
    uint32_t *stu2;  // (candidate pruning) a child list's entries while they are regrouped
    uint32_t *bl;    // the bits of R' (frame bit indices), ascending
    uint32_t *hist;  // counting-sort histogram of a child list
    uint64_t *mR;    // R' words (frame bits)
    uint64_t *Rr;    // R' as positions of N(x) (records)
};

// Candidates [base, base + 64) of frame F: lanes with |R'| = 1 are settled, the
// lanes with |R'| >= 2 are returned.
// IMB: the candidate pruning of section II-C (see heavy_wide); a single-bit candidate whose
// bit is first held by an earlier candidate of the list (a twin, maximal as the first holder)
// left the list with it and is not a node.
// PIV: the pivot rule (see heavy_wide); the candidates the pivot covers, right after it, are
// not taken.
template <bool DIAG, bool ENUM, bool TB, bool IMB = false, bool PIV = false>
__device__ __forceinline__ uint64_t light_wide(const WCtx &w, const FrameState &F, const WFrameView &v, int base,
                                               WaveAcc &acc) {
    const Ctx &c = w.c;
    const int ln = lane_id();
    const int i = base + ln;
    const int nskip = PIV ? (int)uni(*v.skip) : 0;
    const bool act = i < F.n && !(PIV && i > F.nq && i <= F.nq + nskip);
    int r = 0, b = 0;
    if (act)
        for (int q = 0; q < v.wf; ++q) {
            const uint64_t x = v.masks[(size_t)i * v.wf + q];
            if (x) {
                r += __popcll(x);
                b = 64 * q + __ffsll((unsigned long long)x) - 1;
            }
        }
    if (TB && act) acc.dbytes += 8ull * (uint64_t)v.wf;
    if (ENUM) return __ballot(act);
    if (act && r == 1) {
        const bool maximal = v.first[b] == (uint32_t)i;  // no earlier entry holds bit b
        const bool gone = IMB && v.first[b] >= (uint32_t)F.nq && v.first[b] < (uint32_t)i;
        const uint32_t rp = v.orig[b];
        if (maximal) {
            acc.count += 1;
            acc.hash += pair_hash(c.c_is_v, F.sL + v.H[b], c.hvl[rp]);
            acc.out_ints += 2ull + (uint64_t)F.nL + (uint64_t)v.cnt[b] + 1ull;
        }
        if (DIAG && !gone) {
            acc.nodes += 1;
            if (!maximal) acc.nonmax += 1;
            if ((uint32_t)F.level > acc.max_depth) acc.max_depth = (uint32_t)F.level;
            const uint64_t dx = deg_of(c, v.ids[i]);
            const uint64_t rs = 2ull + (uint64_t)c.degl[rp];
            const uint64_t fw = F.fw - (2ull + dx);
            acc.bytes += 4ull * ((2ull + dx) + (rs < fw ? rs : fw) + (uint64_t)(F.n - 1) + 1ull);
        }
        if (TB) acc.dbytes += 8ull + (maximal ? 24ull : 0ull);
    }
    return __ballot(act && r >= 2);
}

// Add a child entry's compressed mask word q (bits 64q ..) to the child's per-bit tables.
__device__ __forceinline__ void wide_table_add(const WFrameView &v2, int q, uint64_t x, uint32_t slot, uint64_t h) {
    while (x) {
        const int t = 64 * q + __ffsll((unsigned long long)x) - 1;
        x &= x - 1ull;
        atomicMin(&v2.first[t], slot);
        atomicAdd(&v2.cnt[t], 1u);
        atomicAdd(reinterpret_cast<unsigned long long *>(&v2.H[t]), (unsigned long long)h);
    }
}

// The candidate at position i of frame F, |R'| >= 2, handled by the whole wave (maximality
// check, expansion, report, child list).
// IMB: the candidate pruning of section II-C.  Candidates of a list are sorted by count, so an
// earlier candidate holding all of a candidate's mask has the same mask (a twin).  When x is
// maximal, its later twins leave the list and join Q with x: a twin whose first twin (the
// earliest) is maximal is never a node, and for the nodes between the two it is a Q entry --
// their child lists take it into Q' instead of P'.  The first twin is maximal exactly when no
// Q entry of the list holds the mask.
// PIV: the pivot pruning of section II-C.  A child list's candidates, sorted by count, are
// regrouped as the pivot p (the first of the largest count), then the candidates whose masks
// lie inside p's (covered: every maximal biclique with one of them holds p), then the rest,
// each group in sorted order; skip[0] of the child frame holds the number covered.  The
// covered ones are never taken: they are candidates for p's node and Q entries (positions
// before) for the nodes after them.
template <bool DIAG, bool ENUM, bool TB, bool IMB = false, bool PIV = false>
__device__ __forceinline__ Node heavy_wide(const WCtx &w, const FrameState &F, const WFrameView &v, int i, FrameState &C,
                                           WaveAcc &acc) {
    const Ctx &c = w.c;
    const int ln = lane_id();
    const uint64_t below = lanes_below();
    const int wf = v.wf;
    // R' (entry i's mask) into the scratch, and its bits in ascending order
    int r = 0;
    for (int q = ln; q < wf; q += 64) {
        const uint64_t x = v.masks[(size_t)i * wf + q];
        w.mR[q] = x;
        r += __popcll(x);
    }
    r = wave_sum_i32(r);
    wait_mem();
    {
        int t0 = 0;
        for (int q = 0; q < wf; ++q) {
            const uint64_t x = uni(w.mR[q]);
            if (!x) continue;
            const bool on = (x >> ln) & 1ull;
            const uint64_t bb = __ballot(on);
            if (on) w.bl[t0 + __popcll(bb & below)] = (uint32_t)(64 * q + ln);
            t0 += __popcll(bb);
        }
        wait_mem();
    }
    if (TB && ln == 0) acc.dbytes += 16ull * (uint64_t)wf + 8ull * (uint64_t)r;

    // maximality: an earlier entry holding all of R' -- a position below i in the AND of R''s
    // rows; a bit of R' first held at i rules that out at once
    bool fh = false;
    for (int t = ln; t < r; t += 64)
        if (v.first[w.bl[t]] == (uint32_t)i) fh = true;
    bool nonmax = false, gone = false;
    if (!__ballot(fh)) {
        const int wl = i >> 6;
        bool inq = false, inp = false;  // (IMB) holders of R' among the Q entries, among earlier candidates
        for (int base = 0; base <= wl && (IMB || !nonmax); base += 64) {
            const int wd = base + ln;
            const bool in = wd <= wl;
            uint64_t a = in ? ~0ull : 0ull;
            int t = 0;
            for (; t < r; ++t) {
                const uint32_t bt = uni(w.bl[t]);
                if (in) a &= v.rows[(size_t)bt * v.nw + wd];
                if ((t & 7) == 7 && !__ballot(a != 0ull)) break;
            }
            if (wd == wl) a &= (1ull << (i & 63)) - 1ull;
            if (__ballot(a != 0ull)) nonmax = true;
            if (IMB) {
                const int q0 = F.nq - 64 * wd;  // positions of word wd below nq
                const uint64_t qm = q0 >= 64 ? ~0ull : (q0 <= 0 ? 0ull : ((1ull << q0) - 1ull));
                inq = inq || (a & qm) != 0ull;
                inp = inp || (a & ~qm) != 0ull;
            }
            if (TB && ln == 0) acc.dbytes += 8ull * (uint64_t)(t < r ? t + 1 : r) * (uint64_t)min(64, wl + 1 - base);
        }
        if (IMB) gone = !__ballot(inq) && __ballot(inp);
    }
    if (gone) return Node::kLeaf;  // left the list with its first twin: not a node
    uint64_t dx = 0, rs = 0;
    if (DIAG) {
        dx = deg_of(c, v.ids[i]);
        uint64_t t2 = 0;
        for (int t = ln; t < r; t += 64) t2 += 2ull + (uint64_t)c.degl[v.orig[w.bl[t]]];
        rs = wave_sum_u64(t2);
        if (ln == 0) {
            acc.nodes += 1;
            if ((uint32_t)F.level > acc.max_depth) acc.max_depth = (uint32_t)F.level;
        }
    }
    if (nonmax) {
        if (DIAG && ln == 0) {
            acc.nonmax += 1;
            const uint64_t fw = F.fw - (2ull + dx);
            acc.bytes += 4ull * ((2ull + dx) + (rs < fw ? rs : fw) + (uint64_t)(F.n - 1) + (uint64_t)r);
        }
        return Node::kLeaf;
    }

    // maximal: per word of positions the OR of R''s rows lists the entries meeting R', the AND
    // those holding all of it (after i; they join L'); the others, Q' before i and P' after,
    // go to stu in list order
    int nu = 0, ne_l = 0, qn_l = 0;
    uint64_t exps = 0;
    {
        const int wi = i >> 6;
        const uint64_t bi = 1ull << (i & 63);
        for (int base = 0; base < v.nw; base += 64) {
            const int wd = base + ln;
            const bool in = wd < v.nw;
            uint64_t u = 0ull, a = in ? ~0ull : 0ull;
            for (int t = 0; t < r; ++t) {
                const uint32_t bt = uni(w.bl[t]);
                if (in) {
                    const uint64_t x = v.rows[(size_t)bt * v.nw + wd];
                    u |= x;
                    a &= x;
                }
            }
            if (wd == wi) {
                u &= ~bi;
                a &= ~bi;
            }
            ne_l += __popcll(a);
            for (uint64_t f = a; f;) {
                const int b = __ffsll((unsigned long long)f) - 1;
                f &= f - 1ull;
                exps += v.hs[64 * wd + b];
            }
            uint64_t qp = u & ~a;
            qn_l += __popcll(qp & (wd < wi ? ~0ull : (wd == wi ? bi - 1ull : 0ull)));
            const int pc = __popcll(qp);
            const int incl = wave_incl_scan(pc);
            int at = nu + incl - pc;
            while (qp) {
                const int b = __ffsll((unsigned long long)qp) - 1;
                qp &= qp - 1ull;
                c.stu[at++] = (uint32_t)(64 * wd + b);
            }
            nu += last_lane(incl);
        }
    }
    int qn = wave_sum_i32(qn_l);
    const int ne = wave_sum_i32(ne_l);
    wait_mem();  // stu is read by other lanes below
    if (IMB) {
        // entries after i that left the list with an earlier twin (of the same count as i, a
        // twin before i, none of the Q entries holding their mask) are Q entries for i: they go
        // to Q' (stu becomes Q' | the moved ones | the rest of P', each in list order)
        const int wl = i >> 6;
        int nmv = 0;
        for (int base = qn; base < nu; base += 64) {
            const int j = base + ln;
            bool mv = false;
            uint32_t k = 0;
            if (j < nu) {
                k = c.stu[j];
                int cnt = 0;
                for (int q = 0; q < wf; ++q) cnt += __popcll(v.masks[(size_t)k * wf + q]);
                if (cnt == r) {
                    bool inq = false, inp = false;
                    for (int wd = 0; wd <= wl; ++wd) {
                        uint64_t a = ~0ull;
                        for (int q = 0; q < wf && a; ++q) {
                            uint64_t x = v.masks[(size_t)k * wf + q];
                            while (x && a) {
                                const int bt = 64 * q + __ffsll((unsigned long long)x) - 1;
                                x &= x - 1ull;
                                a &= v.rows[(size_t)bt * v.nw + wd];
                            }
                        }
                        if (wd == wl) a &= (1ull << (i & 63)) - 1ull;
                        const int q0 = F.nq - 64 * wd;
                        const uint64_t qm = q0 >= 64 ? ~0ull : (q0 <= 0 ? 0ull : ((1ull << q0) - 1ull));
                        inq = inq || (a & qm) != 0ull;
                        inp = inp || (a & ~qm) != 0ull;
                    }
                    mv = inp && !inq;
                }
                c.stu[j] = k | (mv ? 0x80000000u : 0u);  // (positions are below 2^31)
            }
            nmv += __popcll(__ballot(mv));
        }
        if (nmv > 0) {
            wait_mem();
            // stable partition of stu[qn, nu) into the moved entries, then the others
            int am = qn, ak = qn + nmv;
            for (int base = qn; base < nu; base += 64) {
                const int j = base + ln;
                const uint32_t e = j < nu ? c.stu[j] : 0u;
                const bool act = j < nu;
                const bool mv = act && (e & 0x80000000u);
                const uint64_t bm = __ballot(mv), bk = __ballot(act && !mv);
                if (mv) w.stu2[am - qn + __popcll(bm & below)] = e & 0x7FFFFFFFu;
                if (act && !mv) w.stu2[ak - qn + __popcll(bk & below)] = e;
                am += __popcll(bm);
                ak += __popcll(bk);
            }
            wait_mem();
            for (int j = qn + ln; j < nu; j += 64) c.stu[j] = w.stu2[j - qn];
            wait_mem();
            qn += nmv;
        } else {
            for (int j = qn + ln; j < nu; j += 64) c.stu[j] &= 0x7FFFFFFFu;
            wait_mem();
        }
    }
    const int pn = nu - qn;
    // histogram of the P' counts |mask n R'|
    for (int b = ln; b <= r; b += 64) w.hist[b] = 0u;
    wait_mem();
    uint64_t fwc = 0;
    int cmax = 0;  // (PIV) the largest count
    for (int base = 0; base < nu; base += 64) {
        const int j = base + ln;
        if (j < nu) {
            const int k = (int)c.stu[j];
            if (j >= qn) {
                int cnt = 0;
                for (int q = 0; q < wf; ++q) {
                    const uint64_t mq = w.mR[q];
                    if (mq) cnt += __popcll(v.masks[(size_t)k * wf + q] & mq);
                }
                atomicAdd(&w.hist[cnt], 1u);
                if (PIV) cmax = cnt > cmax ? cnt : cmax;
            }
            if (DIAG) fwc += 2ull + deg_of(c, v.ids[k]);
        }
    }
    see_atomics();  // the histogram was built with atomics
    if (TB && ln == 0)
        acc.dbytes += 8ull * (uint64_t)r * (uint64_t)v.nw + 8ull * (uint64_t)ne + 8ull * (uint64_t)nu +
                      (uint64_t)pn * 8ull * (uint64_t)wf + 16ull * (uint64_t)r;

    // report (L', R')
    const uint64_t sL = F.sL + v.hs[i] + wave_sum_u64(exps);
    uint64_t sr = 0;
    for (int t = ln; t < r; t += 64) sr += c.hvl[v.orig[w.bl[t]]];
    sr = wave_sum_u64(sr);
    const int nL = F.nL + 1 + ne;
    if (ln == 0) {
        acc.count += 1;
        acc.hash += pair_hash(c.c_is_v, sL, sr);
        acc.out_ints += 2ull + (uint64_t)nL + (uint64_t)r;
    }
    if (ENUM) {
        for (int q = ln; q < c.Wroot; q += 64) w.Rr[q] = 0ull;
        wait_mem();
        for (int t = ln; t < r; t += 64) {
            const uint32_t rp = v.orig[w.bl[t]];
            atomicOr(reinterpret_cast<unsigned long long *>(&w.Rr[rp >> 6]), 1ull << (rp & 63));
        }
        see_atomics();
        write_record(c, w.Rr, nL, r);
    }
    if (DIAG && ln == 0) {
        const uint64_t fw = F.fw - (2ull + dx);
        acc.bytes += 4ull * ((2ull + dx) + (rs < fw ? rs : fw) + (uint64_t)(F.n - 1) + (uint64_t)r + (uint64_t)pn +
                             (uint64_t)qn);
    }
    if (pn == 0) return Node::kLeaf;

    // child list: Q' in list order, then P' stably sorted by count; masks compressed to the r
    // bits of R' (child bit t = frame bit bl[t]), mapped to N(x) through orig
    const int n2 = nu, wf2 = (r + 63) >> 6;
    const uint32_t off2 = F.top;
    const uint64_t top2 = ((uint64_t)off2 + wframe_words(n2, r) + 1ull) & ~1ull;
    if ((int64_t)top2 > c.scap) {
        if (ln == 0) atomicOr(c.flags, (unsigned int)FLAG_STACK_OVERFLOW);
        return Node::kFull;
    }
    uint32_t *cb = c.stk + off2;
    const WFrameView v2 = wframe_view(cb, n2, r);
    uint32_t *ids2 = cb;
    uint64_t *hs2 = const_cast<uint64_t *>(v2.hs);
    uint64_t *masks2 = const_cast<uint64_t *>(v2.masks);
    int carry = qn;
    for (int base = 0; base <= r; base += 64) {
        const int b = base + ln;
        const int h = b <= r ? (int)w.hist[b] : 0;
        const int incl = wave_incl_scan(h);
        if (b <= r) w.hist[b] = (uint32_t)(carry + incl - h);
        carry += last_lane(incl);
    }
    for (int t = ln; t < r; t += 64) {
        v2.orig[t] = v.orig[w.bl[t]];
        v2.first[t] = kNone;
        v2.cnt[t] = 0u;
        v2.H[t] = 0ull;
    }
    wait_mem();
    const int nbits = r <= 1 ? 1 : 32 - __clz(r - 1);
    if (PIV) {
        // the P' entries in sorted order into stu2 (the placement the plain build makes), then
        // regrouped into stu[qn, nu): the pivot, the entries it covers, the others
        const int cm = __builtin_amdgcn_readfirstlane(wave_max_u32((uint32_t)cmax));
        const int pslot = (int)uni(w.hist[cm]) - qn;  // the first slot of the largest count
        wait_mem();
        for (int base = qn; base < nu; base += 64) {
            const int j = base + ln;
            const bool inp = j < nu;
            const int k = inp ? (int)c.stu[j] : 0;
            int cnt = 0;
            if (inp)
                for (int q = 0; q < wf; ++q) {
                    const uint64_t mq = w.mR[q];
                    if (mq) cnt += __popcll(v.masks[(size_t)k * wf + q] & mq);
                }
            uint64_t same = __ballot(inp);
            for (int bit = 0; bit < nbits; ++bit) {
                const bool on = (cnt >> bit) & 1;
                const uint64_t bb = __ballot(inp && on);
                same &= on ? bb : ~bb;
            }
            uint32_t start = 0;
            if (inp) start = w.hist[cnt];
            if (inp) {
                w.stu2[start + (uint32_t)__popcll(same & below) - (uint32_t)qn] = (uint32_t)k;
                if ((same >> ln) == 1ull) w.hist[cnt] = start + (uint32_t)__popcll(same);
            }
            see_atomics();  // (the next round reads the updated histogram entries; stu2 after)
        }
        const int kp = (int)uni(w.stu2[pslot]);
        int ncov = 0;
        for (int base = 0; base < pn; base += 64) {
            const int t = base + ln;
            bool cov = false;
            if (t < pn && t != pslot) {
                const int k = (int)w.stu2[t];
                cov = true;
                for (int q = 0; q < wf && cov; ++q) {
                    const uint64_t mq = w.mR[q];
                    if (mq) cov = ((v.masks[(size_t)k * wf + q] & mq) & ~v.masks[(size_t)kp * wf + q]) == 0ull;
                }
            }
            if (t < pn) w.stu2[t] |= cov ? 0x80000000u : 0u;  // (positions are below 2^31)
            ncov += __popcll(__ballot(cov));
        }
        wait_mem();
        int ac = qn + 1, ao = qn + 1 + ncov;
        if (ln == 0) c.stu[qn] = (uint32_t)kp;
        for (int base = 0; base < pn; base += 64) {
            const int t = base + ln;
            const bool act = t < pn && t != pslot;
            const uint32_t e = t < pn ? w.stu2[t] : 0u;
            const bool cov = act && (e & 0x80000000u);
            const uint64_t bc = __ballot(cov), bo = __ballot(act && !cov);
            if (cov) c.stu[ac + __popcll(bc & below)] = e & 0x7FFFFFFFu;
            if (act && !cov) c.stu[ao + __popcll(bo & below)] = e;
            ac += __popcll(bc);
            ao += __popcll(bo);
        }
        if (ln == 0) *v2.skip = (uint32_t)ncov;
        wait_mem();
    }
    for (int base = 0; base < nu; base += 64) {
        const int j = base + ln;
        const bool act = j < nu;
        const int k = act ? (int)c.stu[j] : 0;
        const bool inp = !PIV && act && j >= qn;  // (PIV: stu is in its final order)
        int cnt = 0;
        if (inp)
            for (int q = 0; q < wf; ++q) {
                const uint64_t mq = w.mR[q];
                if (mq) cnt += __popcll(v.masks[(size_t)k * wf + q] & mq);
            }
        uint32_t slot = (uint32_t)j;  // Q' entries keep their list order
        if (__ballot(inp)) {
            // stable placement among equal counts: lanes with the same count, in lane order
            uint64_t same = __ballot(inp);
            for (int bit = 0; bit < nbits; ++bit) {
                const bool on = (cnt >> bit) & 1;
                const uint64_t bb = __ballot(inp && on);
                same &= on ? bb : ~bb;
            }
            uint32_t start = 0;
            if (inp) start = w.hist[cnt];
            if (inp) {
                slot = start + (uint32_t)__popcll(same & below);
                if ((same >> ln) == 1ull) w.hist[cnt] = start + (uint32_t)__popcll(same);
            }
            see_atomics();  // (the next round reads the updated histogram entries)
        }
        if (act) {
            ids2[slot] = v.ids[k];
            const uint64_t h = v.hs[k];
            hs2[slot] = h;
            uint64_t ow = 0;
            int t = 0;
            for (int q = 0; q < wf; ++q) {
                uint64_t mq = w.mR[q];
                if (!mq) continue;
                const uint64_t x = v.masks[(size_t)k * wf + q];
                while (mq) {
                    const int p = __ffsll((unsigned long long)mq) - 1;
                    mq &= mq - 1ull;
                    ow |= ((x >> p) & 1ull) << (t & 63);
                    ++t;
                    if ((t & 63) == 0) {
                        masks2[(size_t)slot * wf2 + ((t >> 6) - 1)] = ow;
                        wide_table_add(v2, (t >> 6) - 1, ow, slot, h);
                        ow = 0ull;
                    }
                }
            }
            if (t & 63) {
                masks2[(size_t)slot * wf2 + (t >> 6)] = ow;
                wide_table_add(v2, t >> 6, ow, slot, h);
            }
        }
    }
    see_atomics();
    // position rows: one 64-entry block of one mask word per transpose
    for (int q = 0; q < wf2; ++q)
        for (int blk = 0; blk < v2.nw; ++blk) {
            const int e = 64 * blk + ln;
            const uint64_t t = wave_transpose64(e < n2 ? masks2[(size_t)e * wf2 + q] : 0ull);
            if (64 * q + ln < r) v2.rows[(size_t)(64 * q + ln) * v2.nw + blk] = t;
        }
    wait_mem();
    if (TB && ln == 0)
        acc.dbytes += (uint64_t)n2 * (4ull + 16ull + 8ull * (uint64_t)wf2 + 8ull * (uint64_t)wf) + 32ull * (uint64_t)r +
                      16ull * (uint64_t)r * (uint64_t)n2 / 64ull + 8ull * (uint64_t)r * (uint64_t)v2.nw;
    C.off = off2;
    C.top = (uint32_t)top2;
    C.n = n2;
    C.nq = qn;
    C.level = F.level + 1;
    C.nL = nL;
    C.narrow = 1;
    C.chunk = qn - 64;
    C.rbits = r;
    C.heavy = 0ull;
    C.sL = sL;
    C.fw = DIAG ? wave_sum_u64(fwc) : 0ull;
    return Node::kPushed;
}

// Stable counting sort by key, as wave_sort_by_key, with the histogram in global memory.
template <typename Put>
__device__ __forceinline__ void wave_sort_by_key_g(const uint32_t *src, const uint32_t *key_of, int n, int nbins,
                                                   uint32_t *hist, Put put) {
    const int ln = lane_id();
    const uint64_t below = lanes_below();
    for (int b = ln; b < nbins; b += 64) hist[b] = 0u;
    wait_mem();
    for (int base = 0; base < n; base += 64) {
        const int j = base + ln;
        if (j < n) atomicAdd(&hist[key_of[j]], 1u);
    }
    see_atomics();
    int carry = 0;
    for (int base = 0; base < nbins; base += 64) {
        const int b = base + ln;
        const int h = b < nbins ? (int)hist[b] : 0;
        const int incl = wave_incl_scan(h);
        if (b < nbins) hist[b] = (uint32_t)(carry + incl - h);
        carry += last_lane(incl);
    }
    wait_mem();
    const int nbits = nbins <= 1 ? 1 : 32 - __clz(nbins - 1);
    for (int base = 0; base < n; base += 64) {
        const int j = base + ln;
        const bool act = j < n;
        const uint32_t key = act ? key_of[j] : 0u;
        const uint32_t p = act ? src[j] : 0u;
        uint64_t same = __ballot(act);
        for (int bit = 0; bit < nbits; ++bit) {
            const bool on = (key >> bit) & 1u;
            const uint64_t bb = __ballot(act && on);
            same &= on ? bb : ~bb;
        }
        uint32_t start = 0;
        if (act) start = hist[key];
        if (act) {
            put(start + (uint32_t)__popcll(same & below), p);
            if ((same >> ln) == 1ull) hist[key] = start + (uint32_t)__popcll(same);
        }
        see_atomics();  // (the next round reads the updated histogram entries)
    }
}

// IMB: with the candidate pruning of section II-C (every top-level candidate is searched here
// then): see heavy_wide; at the top level a candidate's twins are the candidates with its exact
// row (a.twin), every first twin is maximal (no earlier candidate can hold its row), and the
// later twins are never nodes.
template <bool DIAG, bool ENUM, bool TB, bool IMB = false, bool PIV = false>
__global__ __launch_bounds__(512) void wide_kernel(SearchArgs a, int64_t lo, int64_t hi, unsigned int *counter) {
    extern __shared__ unsigned char lds_raw[];
    WGShared *sh = reinterpret_cast<WGShared *>(lds_raw);
    const int tid = threadIdx.x, nt = blockDim.x, wid = uni(tid >> 6), nw = nt >> 6, ln = lane_id();
    const WideLayout &L = a.wl;
    const int Wx = L.Wx;
    char *wg = a.warena + (size_t)blockIdx.x * L.wg_bytes;
    uint64_t *bitmap = reinterpret_cast<uint64_t *>(wg + L.off_bitmap);
    uint32_t *bpre = reinterpret_cast<uint32_t *>(wg + L.off_bpre);
    uint64_t *M = reinterpret_cast<uint64_t *>(wg + L.off_M);
    int32_t *gid = reinterpret_cast<int32_t *>(wg + L.off_gid);
    uint32_t *cnt1 = reinterpret_cast<uint32_t *>(wg + L.off_cnt);
    uint64_t *hvl = reinterpret_cast<uint64_t *>(wg + L.off_hv);
    uint32_t *degl = reinterpret_cast<uint32_t *>(wg + L.off_deg);
    uint32_t *t1v = reinterpret_cast<uint32_t *>(wg + L.off_t1v);
    uint32_t *t1c = reinterpret_cast<uint32_t *>(wg + L.off_t1c);
    uint32_t *whist = reinterpret_cast<uint32_t *>(wg + L.off_whist);
    uint32_t *s1 = reinterpret_cast<uint32_t *>(wg + L.off_S1);
    char *wv = wg + L.off_waves + (size_t)wid * L.wave_bytes;
    FrameState *hdr = reinterpret_cast<FrameState *>(wv + L.off_w_hdr);

    WCtx w;
    Ctx &c = w.c;
    c.gid = gid;
    c.M = M;
    c.hvl = hvl;
    c.degl = degl;
    c.c_off = a.c_off;
    c.s1 = s1;
    c.stk = reinterpret_cast<uint32_t *>(wv + L.off_w_stack);
    c.stu = reinterpret_cast<uint32_t *>(wv + L.off_w_u);
    c.scap = L.scap;
    c.c_is_v = 0;
    c.cbase = 0;
    c.obase = 0;
    c.Wroot = Wx;
    c.rec = a.rec;
    c.rec_cap = a.rec_cap;
    c.rec_offs = a.rec_offs;
    c.rec_offs_cap = a.rec_offs_cap;
    c.rec_batch = a.rec_batch;
    c.res = nullptr;
    c.acc = a.acc;
    c.flags = a.flags;
    w.stu2 = reinterpret_cast<uint32_t *>(wv + L.off_w_u2);
    w.bl = reinterpret_cast<uint32_t *>(wv + L.off_w_bl);
    w.hist = reinterpret_cast<uint32_t *>(wv + L.off_w_hist);
    w.mR = reinterpret_cast<uint64_t *>(wv + L.off_w_mr);
    w.Rr = reinterpret_cast<uint64_t *>(wv + L.off_w_rr);

    WaveAcc acc{};
    const uint64_t ld_start = TB ? wall_clock64() : 0ull;
    const int ucap = a.dims.ucap;
    const int64_t nroots = hi - lo;
    const int64_t ntasks = nroots * (int64_t)L.reps;
    if (tid < 16) sh->red[tid] = 0ull;
    if (tid == 0) sh->graph = -1;
    __syncthreads();

    for (;;) {
        if (tid == 0) {
            const unsigned int f = __hip_atomic_load(a.flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            unsigned long long t = (f & FLAG_RERUN) ? ~0ull : (unsigned long long)atomicAdd(counter, 1u);
            while (t != ~0ull && (int64_t)t < ntasks && root_cancelled(a, lo + (int64_t)t % nroots))
                t = (unsigned long long)atomicAdd(counter, 1u);
            sh->task = t;
        }
        __syncthreads();
        const unsigned long long tt = sh->task;
        if (tt == ~0ull || (int64_t)tt >= ntasks) break;
        const int64_t ri = (int64_t)tt % nroots;   // top-level candidates of largest degree first
        const bool owner = (int64_t)tt < nroots;   // replica 0 reports the top-level node
        int g = 0;
        int64_t k;
        if (a.tasks) {
            const unsigned long long tk = a.tasks[lo + ri];
            g = (int)(tk >> 32);
            k = (int64_t)(tk & 0xFFFFFFFFull);
        } else {
            k = hi - 1 - ri;
        }
        if (g != sh->graph) {
            if (sh->graph >= 0) flush_acc<DIAG, TB>(acc, a.graphs[sh->graph].acc, sh);
            __syncthreads();
            if (tid == 0) sh->graph = g;
            __syncthreads();
        }
        const GraphDesc gd = a.graphs[g];
        c.c_is_v = gd.c_is_v;
        c.cbase = gd.cbase;
        c.obase = gd.obase;
        const int nwords = gd.nwords;
        const int32_t x = gd.order[k];
        const int32_t rbx = a.c_off[x];
        const int32_t d = a.c_off[x + 1] - rbx;
        const int32_t *row = a.c_adj + rbx;
        c.row = row;
        c.x_root = x;
        const int wd = (d + 63) >> 6;

        // -- reverse scan 1: mark the ranks of all 2-hop neighbours of x
        for (int j = wid; j < d; j += nw) {
            const int32_t wv2 = row[j];
            const int32_t e0 = a.o_off[wv2], e1 = a.o_off[wv2 + 1];
            for (int p = e0 + ln; p < e1; p += 64) {
                const int32_t v = a.o_adj[p];
                if (v != x) {
                    const int32_t rk = a.rank[v];
                    atomicOr(reinterpret_cast<unsigned long long *>(&bitmap[rk >> 6]), 1ull << (rk & 63));
                }
            }
        }
        uint64_t hv_local = 0, rs_local = 0;
        for (int j = tid; j < d; j += nt) {
            const int32_t wv2 = row[j];
            const uint64_t h = hr(c, wv2);
            hvl[j] = h;
            hv_local += h;
            const uint32_t dw = (uint32_t)(a.o_off[wv2 + 1] - a.o_off[wv2]);
            degl[j] = dw;
            rs_local += 2ull + dw;
        }
        if (tid == 0) {
            sh->nonmax = 0;
            sh->pcount = 0;
            sh->exps = 0;
            sh->fw1 = 0;
            sh->hvsum = 0;
            sh->rs1 = 0;
            sh->nexp = 0;
        }
        __syncthreads();
        see_atomics();
        hv_local = wave_sum_u64(hv_local);
        rs_local = wave_sum_u64(rs_local);
        if (ln == 0) {
            lds_add(&sh->hvsum, hv_local);
            lds_add(&sh->rs1, rs_local);
        }
        block_popcount_prefix(bitmap, bpre, nwords, sh);
        const int s0 = uni(sh->s0);
        if (s0 > ucap) {
            for (int q = tid; q < nwords; q += nt) bitmap[q] = 0ull;
            if (tid == 0) {
                atomicOr(a.flags, (unsigned int)FLAG_UNIVERSE_OVERFLOW);
                atomicMax(&a.acc[ACC_NEED_UCAP], (unsigned long long)s0);
            }
            __syncthreads();
            continue;
        }
        const int nq0 = (int)bpre[k >> 6] + __popcll(bitmap[k >> 6] & ((1ull << (k & 63)) - 1ull));
        c.s0 = s0;
        for (int q = tid; q < nwords; q += nt) {
            uint64_t bits = bitmap[q];
            uint32_t pos = bpre[q];
            while (bits) {
                const int b = __ffsll((unsigned long long)bits) - 1;
                bits &= bits - 1ull;
                gid[pos++] = gd.order[q * 64 + b];
            }
        }
        for (size_t q = tid; q < (size_t)s0 * Wx; q += nt) M[q] = 0ull;
        wait_mem();
        __syncthreads();
        // -- reverse scan 2: M[v] gets bit j for every w_j in N(x) adjacent to v
        for (int j = wid; j < d; j += nw) {
            const int32_t wv2 = row[j];
            const int32_t e0 = a.o_off[wv2], e1 = a.o_off[wv2 + 1];
            for (int p = e0 + ln; p < e1; p += 64) {
                const int32_t v = a.o_adj[p];
                if (v != x) {
                    const int32_t rk = a.rank[v];
                    const uint32_t li =
                        bpre[rk >> 6] + (uint32_t)__popcll(bitmap[rk >> 6] & ((1ull << (rk & 63)) - 1ull));
                    atomicOr(reinterpret_cast<unsigned long long *>(&M[(size_t)li * Wx + (j >> 6)]), 1ull << (j & 63));
                }
            }
        }
        __syncthreads();
        see_atomics();
        for (int q = tid; q < nwords; q += nt) bitmap[q] = 0ull;
        // -- the top-level node for x: counts, maximality against earlier ranks, expansion
        {
            bool nm = false;
            int pc = 0, nexp = 0;
            uint64_t ex = 0, fw = 0;
            for (int li = tid; li < s0; li += nt) {
                int cc = 0;
                for (int q = 0; q < wd; ++q) cc += __popcll(M[(size_t)li * Wx + q]);
                cnt1[li] = (uint32_t)cc;
                const int32_t gv = gid[li];
                const uint64_t dg = DIAG ? 2ull + (uint64_t)(a.c_off[gv + 1] - a.c_off[gv]) : 0ull;
                if (li < nq0) {
                    if (cc == d) nm = true;
                    else fw += dg;
                } else if (cc == d) {
                    ex += hl(c, gv);
                    ++nexp;
                } else {
                    ++pc;
                    fw += dg;
                }
            }
            if (__ballot(nm) && ln == 0) atomicOr(&sh->nonmax, 1);
            ex = wave_sum_u64(ex);
            fw = wave_sum_u64(fw);
            pc = wave_sum_i32(pc);
            nexp = wave_sum_i32(nexp);
            if (ln == 0) {
                atomicAdd(&sh->pcount, pc);
                atomicAdd(&sh->nexp, nexp);
                lds_add(&sh->exps, ex);
                lds_add(&sh->fw1, fw);
            }
        }
        wait_mem();
        __syncthreads();
        const bool root_nonmax = uni(sh->nonmax) != 0;
        const int P1 = uni(sh->pcount);
        if (tid == 0 && owner) {
            const uint64_t dx = (uint64_t)d;
            // (IMB: a top-level candidate with an earlier twin is exactly a non-maximal one,
            // and it left the list with its first twin: not a node)
            if (DIAG && !(IMB && root_nonmax)) {
                acc.nodes += 1;
                if (acc.max_depth < 1) acc.max_depth = 1;
                const uint64_t fwtop = gd.total_fw - (2ull + dx);
                const uint64_t rs = sh->rs1;
                uint64_t b = (2ull + dx) + (rs < fwtop ? rs : fwtop) + (uint64_t)(gd.ncand - 1) + dx;
                if (root_nonmax) acc.nonmax += 1;
                else b += (uint64_t)P1 + (uint64_t)nq0;
                acc.bytes += 4ull * b;
            }
            if (TB) {
                const uint64_t wk = (uint64_t)sh->rs1 - 2ull * dx, su = (uint64_t)s0;
                acc.dbytes += 4ull * (dx + 2ull) + 16ull * dx + 44ull * wk + 12ull * dx + 32ull * (uint64_t)nwords +
                              8ull * su + 16ull * (uint64_t)wd * su + 8ull * su;
            }
            if (!root_nonmax) {
                acc.count += 1;
                acc.hash += pair_hash(c.c_is_v, hl(c, x) + sh->exps, sh->hvsum);
                acc.out_ints += 2ull + (uint64_t)(1 + sh->nexp) + (uint64_t)d;
            }
        }
        if (ENUM && !root_nonmax && owner && wid == 0) {
            for (int q = ln; q < Wx; q += 64) {
                const int bits = d - 64 * q;
                w.Rr[q] = bits >= 64 ? ~0ull : (bits <= 0 ? 0ull : ((1ull << bits) - 1ull));
            }
            wait_mem();
            write_record(c, w.Rr, 1 + sh->nexp, d);
        }
        if (root_nonmax || P1 == 0) {
            __syncthreads();
            continue;
        }
        // -- the top-level list as a frame: Q1 (earlier ranks) ++ P1 stably sorted by count,
        //    masks over the positions of N(x), per-bit tables, rows
        const int n1 = nq0 + P1;
        const WFrameView v1 = wframe_view(s1, n1, d);
        uint32_t *ids1 = s1;
        for (int li = tid; li < nq0; li += nt) ids1[li] = (uint32_t)li;
        if (wid == 0) {
            // (IMB) candidates ranked after x with a twin ranked before x left the list with it:
            // they join Q1, after the earlier ranks, in rank order
            int pn = 0, nmv = 0;
            for (int base = nq0; base < s0; base += 64) {
                const int li = base + ln;
                const bool act2 = li < s0;
                const uint32_t cc = act2 ? cnt1[li] : 0u;
                const bool cand = act2 && (int)cc < d;
                const bool mv = IMB && cand && a.twin[gid[li]] < (int32_t)k;
                const bool pk = cand && !mv;
                const uint64_t pb = __ballot(pk), mb = __ballot(mv);
                if (pk) {
                    const int p = pn + __popcll(pb & lanes_below());
                    t1v[p] = (uint32_t)li;
                    t1c[p] = cc;
                }
                if (mv) ids1[nq0 + nmv + __popcll(mb & lanes_below())] = (uint32_t)li;
                pn += __popcll(pb);
                nmv += __popcll(mb);
            }
            if (ln == 0) sh->pcount = pn;  // the candidates left in the list
            wait_mem();
            const int q1 = nq0 + nmv;
            wave_sort_by_key_g(t1v, t1c, pn, d, whist, [&](uint32_t slot, uint32_t li) { ids1[q1 + slot] = li; });
            if (PIV) {
                // (PIV) regrouped: the pivot (the first of the largest count), the candidates
                // whose masks lie inside its mask, the others; t1v is free after the sort
                wait_mem();
                const uint32_t cm = cnt1[uni(ids1[q1 + pn - 1])];
                int nmax = 0;
                for (int base = 0; base < pn; base += 64) {
                    const int t = base + ln;
                    nmax += __popcll(__ballot(t < pn && cnt1[ids1[q1 + t]] == cm));
                }
                const int pslot = pn - nmax;
                const uint32_t lp = uni(ids1[q1 + pslot]);
                int ncov = 0;
                for (int base = 0; base < pn; base += 64) {
                    const int t = base + ln;
                    bool cov = false;
                    uint32_t li = 0;
                    if (t < pn) li = ids1[q1 + t];
                    if (t < pn && t != pslot) {
                        cov = true;
                        for (int q = 0; q < wd && cov; ++q)
                            cov = (M[(size_t)li * Wx + q] & ~M[(size_t)lp * Wx + q]) == 0ull;
                    }
                    if (t < pn) t1v[t] = li | (cov ? 0x80000000u : 0u);  // (indices are below 2^31)
                    ncov += __popcll(__ballot(cov));
                }
                wait_mem();
                int ac = 1, ao = 1 + ncov;
                if (ln == 0) ids1[q1] = lp;
                for (int base = 0; base < pn; base += 64) {
                    const int t = base + ln;
                    const bool act = t < pn && t != pslot;
                    const uint32_t e = t < pn ? t1v[t] : 0u;
                    const bool cov = act && (e & 0x80000000u);
                    const uint64_t bc = __ballot(cov), bo = __ballot(act && !cov);
                    if (cov) ids1[q1 + ac + __popcll(bc & lanes_below())] = e & 0x7FFFFFFFu;
                    if (act && !cov) ids1[q1 + ao + __popcll(bo & lanes_below())] = e;
                    ac += __popcll(bc);
                    ao += __popcll(bo);
                }
                if (ln == 0) *v1.skip = (uint32_t)ncov;
                wait_mem();
            }
        }
        for (int b = tid; b < d; b += nt) {
            v1.first[b] = kNone;
            v1.cnt[b] = 0u;
            v1.H[b] = 0ull;
            v1.orig[b] = (uint32_t)b;
        }
        wait_mem();
        __syncthreads();
        uint64_t *masks1 = const_cast<uint64_t *>(v1.masks);
        uint64_t *hs1 = const_cast<uint64_t *>(v1.hs);
        for (int j = tid; j < n1; j += nt) {
            const uint32_t li = ids1[j];
            const uint64_t h = hl(c, gid[li]);
            hs1[j] = h;
            for (int q = 0; q < wd; ++q) {
                uint64_t mm = M[(size_t)li * Wx + q];
                masks1[(size_t)j * wd + q] = mm;
                while (mm) {
                    const int b = 64 * q + __ffsll((unsigned long long)mm) - 1;
                    mm &= mm - 1ull;
                    atomicMin(&v1.first[b], (uint32_t)j);
                    atomicAdd(&v1.cnt[b], 1u);
                    atomicAdd(reinterpret_cast<unsigned long long *>(&v1.H[b]), (unsigned long long)h);
                }
            }
        }
        __syncthreads();
        see_atomics();
        for (int job = wid; job < v1.nw * wd; job += nw) {
            const int blk = job / wd, q = job - blk * wd;
            const int e = 64 * blk + ln;
            const uint64_t t = wave_transpose64(e < n1 ? masks1[(size_t)e * wd + q] : 0ull);
            if (64 * q + ln < d) v1.rows[(size_t)(64 * q + ln) * v1.nw + blk] = t;
        }
        wait_mem();
        __syncthreads();
        if (TB && tid == 0 && owner)
            acc.dbytes += 4ull * (uint64_t)nq0 + 4ull * (uint64_t)(s0 - nq0) + 20ull * (uint64_t)P1 +
                          (uint64_t)n1 * (24ull + 16ull * (uint64_t)wd) + 32ull * (uint64_t)d +
                          8ull * (uint64_t)n1 * (uint64_t)wd + 8ull * (uint64_t)d * (uint64_t)v1.nw;

        const int P1c = IMB ? uni(sh->pcount) : P1;  // candidates of the list
        FrameState top;
        top.off = kShared;
        top.top = 0;
        top.n = n1;
        top.nq = n1 - P1c;
        top.level = 2;
        top.nL = 1 + uni(sh->nexp);
        top.narrow = 1;
        top.chunk = 0;
        top.rbits = d;
        top.heavy = 0ull;
        top.sL = hl(c, x) + uni((uint64_t)sh->exps);
        top.fw = uni((uint64_t)sh->fw1);
        const int nch = (P1c + 63) >> 6;

        // -- chunks of the top-level list, claimed by every wave of every replica; each wave
        //    searches depth-first below the candidates of its chunk
        bool aborted = false;
        for (;;) {
            int q = 0;
            if (ln == 0) q = (int)atomicAdd(&a.wide_items[ri], 1u);
            q = __builtin_amdgcn_readlane(q, 0);
            if (q >= nch) break;
            if (uni(__hip_atomic_load(a.flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) & FLAG_RERUN) break;
            FrameState cur = top;
            cur.chunk = top.nq + 64 * q;
            cur.heavy = light_wide<DIAG, ENUM, TB, IMB, PIV>(w, cur, v1, cur.chunk, acc);
            int depth = 0;
            while (!aborted) {
                const WFrameView v = wframe_view(frame_base(c, cur.off), cur.n, cur.rbits);
                if (cur.heavy == 0ull) {
                    if (depth == 0) break;  // the chunk is done
                    const int base = cur.chunk + 64;
                    if (base >= cur.n) {
                        --depth;
                        cur = uni_frame(hdr[depth]);
                        continue;
                    }
                    cur.chunk = base;
                    cur.heavy = light_wide<DIAG, ENUM, TB, IMB, PIV>(w, cur, v, base, acc);
                    continue;
                }
                const int lane = __ffsll((unsigned long long)cur.heavy) - 1;
                cur.heavy &= cur.heavy - 1ull;
                FrameState ch;
                const Node node = heavy_wide<DIAG, ENUM, TB, IMB, PIV>(w, cur, v, cur.chunk + lane, ch, acc);
                if (node == Node::kPushed) {
                    if (depth + 1 >= L.maxdepth) {
                        if (ln == 0) atomicOr(a.flags, (unsigned int)FLAG_DEPTH_OVERFLOW);
                        aborted = true;
                        break;
                    }
                    hdr[depth] = cur;  // every lane stores the same header
                    wait_mem();
                    if (TB && ln == 0) acc.dbytes += 2ull * sizeof(FrameState);
                    ++depth;
                    cur = ch;
                } else if (node == Node::kFull || stack_ran_out(a.flags)) {
                    aborted = true;
                }
            }
            if (aborted) break;
        }
        __syncthreads();
    }
    if (sh->graph >= 0) flush_acc<DIAG, TB>(acc, a.graphs[sh->graph].acc, sh);
    if (TB && a.wg_load && tid == 0) {
        a.wg_load[3 * (size_t)blockIdx.x] = ld_start;
        a.wg_load[3 * (size_t)blockIdx.x + 1] = wall_clock64();
        a.wg_load[3 * (size_t)blockIdx.x + 2] = 0ull;  // replicas take chunks without waiting
    }
}

size_t lds_bytes(int W, int waves, int nwords) {
    return sizeof(WGShared) + hist_region_bytes(64 * W, waves) + (size_t)waves * kWaveLds + rank_lds_bytes(nwords);
}

template <int W>
hipError_t launch_w(const SearchArgs &a, bool diag, bool enumerate, bool tb, int64_t lo, int64_t hi, unsigned int *counter,
                    int grid, int waves, hipStream_t s) {
    dim3 g(grid), b(64 * waves);
    const size_t lds = lds_bytes(W, waves, a.dims.nwords);
    if (tb && !diag && !enumerate)
        hipLaunchKernelGGL((search_kernel<W, false, false, true>), g, b, lds, s, a, lo, hi, counter);
    else if (diag && enumerate)
        hipLaunchKernelGGL((search_kernel<W, true, true>), g, b, lds, s, a, lo, hi, counter);
    else if (diag)
        hipLaunchKernelGGL((search_kernel<W, true, false>), g, b, lds, s, a, lo, hi, counter);
    else if (enumerate)
        hipLaunchKernelGGL((search_kernel<W, false, true>), g, b, lds, s, a, lo, hi, counter);
    else
        hipLaunchKernelGGL((search_kernel<W, false, false>), g, b, lds, s, a, lo, hi, counter);
    return hipGetLastError();
}

size_t align_up(size_t x, size_t al) { return (x + al - 1) / al * al; }

template <int W, bool DIAG, bool ENUM>
int occ(int waves, int nwords) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, search_kernel<W, DIAG, ENUM>, 64 * waves,
                                                      lds_bytes(W, waves, nwords)) != hipSuccess)
        return 2;
    return nb > 0 ? nb : 1;
}

template <int W>
int occ_w(bool diag, bool enumerate, int waves, int nwords) {
    if (diag && enumerate) return occ<W, true, true>(waves, nwords);
    if (diag) return occ<W, true, false>(waves, nwords);
    if (enumerate) return occ<W, false, true>(waves, nwords);
    return occ<W, false, false>(waves, nwords);
}

}  // namespace

int search_occupancy(int W, bool diag, bool enumerate, int waves, int nwords) {
    switch (W) {
        case 1: return occ_w<1>(diag, enumerate, waves, nwords);
        case 2: return occ_w<2>(diag, enumerate, waves, nwords);
        case 4: return occ_w<4>(diag, enumerate, waves, nwords);
        case 8: return occ_w<8>(diag, enumerate, waves, nwords);
        default: return occ_w<16>(diag, enumerate, waves, nwords);
    }
}

WideLayout wide_layout(const SearchDims &d, int Wx, int64_t scap, int32_t maxdepth, int waves) {
    WideLayout L{};
    L.Wx = Wx;
    L.scap = scap;
    L.maxdepth = maxdepth;
    const size_t ucap = (size_t)d.ucap, W = (size_t)Wx, bits = 64 * W;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o = align_up(o + bytes, 256);
        return at;
    };
    L.off_bitmap = take((size_t)d.nwords * 8);
    L.off_bpre = take(((size_t)d.nwords + 1) * 4);
    L.off_M = take(ucap * W * 8);
    L.off_gid = take(ucap * 4);
    L.off_cnt = take(ucap * 4);
    L.off_hv = take(bits * 8);
    L.off_deg = take(bits * 4);
    L.off_t1v = take(ucap * 4);
    L.off_t1c = take(ucap * 4);
    L.off_whist = take((bits + 1) * 4);
    // the top-level list: ids | hs | masks | first, cnt | H | orig | rows (see wframe_view)
    const size_t s1_words = align_up(ucap, 2) + 2 * ucap + 2 * ucap * W + 4 * bits + bits + 2 + 2 * bits * ((ucap + 63) / 64) + 2;
    L.off_S1 = take(s1_words * 4);
    L.off_waves = o;
    size_t w = 0;
    auto wtake = [&](size_t bytes) {
        const size_t at = w;
        w = align_up(w + bytes, 256);
        return at;
    };
    L.off_w_stack = wtake((size_t)scap * 4);
    L.off_w_u = wtake(ucap * 4);
    L.off_w_u2 = wtake(ucap * 4);
    L.off_w_bl = wtake(bits * 4);
    L.off_w_hist = wtake((bits + 2) * 4);
    L.off_w_mr = wtake(W * 8);
    L.off_w_rr = wtake(W * 8);
    L.off_w_hdr = wtake((size_t)maxdepth * sizeof(FrameState));
    L.wave_bytes = w;
    L.wg_bytes = align_up(o + (size_t)waves * w, 4096);
    return L;
}

hipError_t launch_wide(const SearchArgs &a, bool diag, bool enumerate, bool tb, int64_t lo, int64_t hi,
                       unsigned int *counter, int grid, int waves, hipStream_t s, int prune) {
    dim3 g(grid), b(64 * waves);
    const size_t lds = sizeof(WGShared);
    if (prune == 2) {
        if (enumerate)
            hipLaunchKernelGGL((wide_kernel<false, true, false, false, true>), g, b, lds, s, a, lo, hi, counter);
        else if (diag)
            hipLaunchKernelGGL((wide_kernel<true, false, false, false, true>), g, b, lds, s, a, lo, hi, counter);
        else
            hipLaunchKernelGGL((wide_kernel<false, false, false, false, true>), g, b, lds, s, a, lo, hi, counter);
        return hipGetLastError();
    }
    if (prune == 1) {
        if (enumerate)
            hipLaunchKernelGGL((wide_kernel<false, true, false, true>), g, b, lds, s, a, lo, hi, counter);
        else if (diag)
            hipLaunchKernelGGL((wide_kernel<true, false, false, true>), g, b, lds, s, a, lo, hi, counter);
        else
            hipLaunchKernelGGL((wide_kernel<false, false, false, true>), g, b, lds, s, a, lo, hi, counter);
        return hipGetLastError();
    }
    if (tb && !diag && !enumerate)
        hipLaunchKernelGGL((wide_kernel<false, false, true>), g, b, lds, s, a, lo, hi, counter);
    else if (diag && enumerate)
        hipLaunchKernelGGL((wide_kernel<true, true, false>), g, b, lds, s, a, lo, hi, counter);
    else if (diag)
        hipLaunchKernelGGL((wide_kernel<true, false, false>), g, b, lds, s, a, lo, hi, counter);
    else if (enumerate)
        hipLaunchKernelGGL((wide_kernel<false, true, false>), g, b, lds, s, a, lo, hi, counter);
    else
        hipLaunchKernelGGL((wide_kernel<false, false, false>), g, b, lds, s, a, lo, hi, counter);
    return hipGetLastError();
}

ArenaLayout search_layout(const SearchDims &d) {
    ArenaLayout L{};
    const size_t ucap = (size_t)d.ucap, W = (size_t)d.Wmax, bits = 64 * W;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o = align_up(o + bytes, 256);
        return at;
    };
    L.off_bitmap = take((size_t)d.nwords * 8);
    L.off_bpre = take(((size_t)d.nwords + 1) * 4);
    L.off_M = take(ucap * W * 8);
    L.off_gid = take(ucap * 4);
    L.off_cnt = take(ucap * 4);
    L.off_hv = take(bits * 8);
    L.off_deg = take(bits * 4);
    L.off_t1v = take(ucap * 4);
    // (the staged counts are used while the top-level list is built, its record only after that)
    static_assert(sizeof(TopRec) <= 256, "the record fits the smallest region");
    L.off_top = L.off_t1c = take(ucap * 4);
    // ids | hs | masks | first, cnt | H | orig | rows (see frame_view)
    L.s1_words = align_up(ucap, 2) + 2 * ucap + 2 * ucap * W + 2 * bits + 2 * bits + 64 + 128 + 2 * bits * ((ucap + 63) / 64) + 2;
    L.off_S1 = take(L.s1_words * 4);
    L.off_hb = take((ucap / 64 + 1) * 8);
    L.off_hpre = take((ucap / 64 + 2) * 4);
    L.off_hpos = take(ucap * 4);
    L.off_waves = o;
    size_t w = 0;
    auto wtake = [&](size_t bytes) {
        const size_t at = w;
        w = align_up(w + bytes, 256);
        return at;
    };
    L.off_w_stack = wtake((size_t)d.scap * 4);
    L.off_w_u = wtake(ucap * 4);
    L.off_w_hdr = wtake((size_t)d.maxdepth * sizeof(FrameState));
    L.wave_bytes = w;
    L.wg_bytes = align_up(o + (size_t)d.waves * w, 4096);
    return L;
}

hipError_t launch_search(const SearchArgs &a, int W, bool diag, bool enumerate, bool tb, int64_t lo, int64_t hi,
                         unsigned int *counter, int grid, int waves, hipStream_t s) {
    switch (W) {
        case 1: return launch_w<1>(a, diag, enumerate, tb, lo, hi, counter, grid, waves, s);
        case 2: return launch_w<2>(a, diag, enumerate, tb, lo, hi, counter, grid, waves, s);
        case 4: return launch_w<4>(a, diag, enumerate, tb, lo, hi, counter, grid, waves, s);
        case 8: return launch_w<8>(a, diag, enumerate, tb, lo, hi, counter, grid, waves, s);
        case 16: return launch_w<16>(a, diag, enumerate, tb, lo, hi, counter, grid, waves, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace mbe
