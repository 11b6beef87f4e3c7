#pragma once
// k-way sparse union addition (and intersection product): assembly (count),
// prefix sum and compute (fill) of Section 4.3 / 4.4 (pipeline of Figure 7(a))
// in ONE kernel, one workgroup of eight wavefronts per partition.
//
// A partition owns, in every operand t, the stored entries at last-level
// positions [q_t(p), q_t(p+1)) found by the partition search; because the
// search runs in coordinate space, entries with equal coordinates in different
// operands always fall in the same partition (Section 6, merge-path paragraph),
// so a partition's output is independent of its neighbours: there is no carry.
//
// Per partition the workgroup
//   1. stages the KEYS of its entries in LDS as k sorted runs, each followed by a
//      sentinel: the stored coordinates are copied by the memory pipeline itself
//      (16 bytes per lane, no register in between); for vectors they are the keys.
//      Matrices and tensors: key = row field above column field, the row counted
//      from the partition's first one, so that the key of practically every
//      partition fits 32 bits; the row of an entry comes from a bit per row start
//      (set from the pos arrays) and the latest set bit at or before the entry;
//   2. merges the runs pairwise.  Every thread owns R consecutive places of the
//      merged order, finds where they start with a diagonal search (the search of
//      Section 3.2 on two one-level operands) and merges them serially without
//      branches.  What comes out of the last merge is the ORDER -- a 16-bit word
//      per place that names operand and staged word of its entry -- and one bit
//      per place that says whether its key differs from the one before it (a HEAD),
//      one whether its row does;
//   3. assembly: the heads are the output entries of the union, the heads that
//      k - 1 equal keys follow those of the product; every wavefront counts all
//      bits by itself (two 64-bit words per lane and one scan);
//   4. prefix sum: publishes the partition's counts, then (sums) every thread asks
//      for the VALUES of its output entries, straight from the operands: in the
//      merged order a wavefront's 64 places read one contiguous stretch per
//      operand, and the values need no place in LDS; products multiply theirs
//      here.  Behind the values come the counts of everything before the
//      partition (two levels, see below);
//   5. compute: every output entry writes coordinate and value at offset + heads
//      before it -- consecutive lanes write consecutive words.  The hierarchical
//      arrays (crd0/pos1 of a DCSR result, pos of a CSR result, crd1/pos2 and
//      crd0/pos1 of a third-order result) are written for the rows (fibres,
//      slices) whose first output entry the partition owns -- exactly one
//      writer each.
// What differs from the paper's three kernels: the inputs are read once instead
// of twice and there is no separate scan launch; the arithmetic is the same.
//
// What bounds it, and why it is cut like this: a partition is a chain of latencies
// (table, entries, LDS merge, counts of the predecessors, stores), so what counts
// is how many entries are in flight per compute unit and how short the chain is.
// With 6 bytes of LDS per entry and 64 registers four workgroups of up to 5544
// entries run on a compute unit (the form before it kept 8-byte keys and the
// values in LDS: three workgroups of 3556), and the chain has five barriers
// instead of sixteen.
//
// Workgroup p handles partition p and waits, when it looks up its offset, only
// for workgroups with a smaller index.  Workgroups are handed to every XCD in
// index order, so the unfinished workgroup with the smallest index is always
// running and waits for nobody: the waits end.  (Every wait is bounded all the
// same; a wavefront that gives up reports NACHO_ERR_HIP and writes nothing.)
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"
#include "search.hpp"

namespace nacho {

namespace {

#ifndef NACHO_MERGE_WAVES
#define NACHO_MERGE_WAVES 8
#endif
constexpr int kWaves = NACHO_MERGE_WAVES;           // wavefronts per workgroup
constexpr int kThreads = kWaves * NACHO_WAVE;
constexpr int kMaxRuns = NACHO_MAX_OPERANDS;

// Places of the merged order a thread owns.  Odd where it can be: thread i's places start at word
// i * kIpt of the LDS arrays, and an odd stride spreads the lanes of a wavefront
// over all banks (ten: two lanes a bank).  Large calls: chosen so that four workgroups fit a compute unit: its
// LDS (6 bytes per entry with 32-bit keys, 10 with 64-bit ones) and, values of 8 bytes,
// the registers that hold a thread's values while the prefix sum is looked up.  Calls of one
// round of workgroups: a thread's serial share is what such a call takes, so it is short (merge_fields has
// the lines).  Remapped operands have at most 4096 entries a partition, which nine places a thread hold: with
// eleven two of eight wavefronts had nothing to do (the product of two DCSR matrices of 20M 166 to 155.5 us).
// Twelve for 32-bit values: two DCSR matrices of 20M 157 to 154 us, but three vectors 61.7 to 63.4.
template <typename KeyT, typename T, int kSize> struct Shape {
    static constexpr int kIpt = kSize == MERGE_SHORT ? 3 : (sizeof(KeyT) == 8 ? 7 : (kSize == MERGE_MIDDLE ? 9 : (sizeof(T) == 8 ? 10 : 11)));
    static constexpr int kTile = kThreads * kIpt;
    // Entries a partition may hold.  A run occupies up to seven words besides its entries (up to three
    // before it: the copy starts on a 16-byte boundary; its sentinel; the next run's alignment) and the
    // runs start at word 4; every round of pairwise merges hands out whole threads per pair.
    static constexpr int kCapacity = kTile - 8 * kMaxRuns > kIpt * (kThreads - kMaxRuns)
                                         ? kIpt * (kThreads - kMaxRuns) : kTile - 8 * kMaxRuns;
    static constexpr int kBlocks = kTile / NACHO_WAVE;     // blocks of 64 places
    static constexpr int kWords = kTile + 48;              // (a thread past the last place reads on)
    static_assert(kBlocks <= 2 * NACHO_WAVE, "a lane holds the bits of two blocks");
    static_assert(kTile <= (1 << 13), "the word of an entry fits 13 bits of its order word");
};

// Prefix sum over the workgroups' counts, two levels and no chains: a workgroup
// publishes the counts of its partition in a 32-bit word; the last workgroup
// of every chunk of kChunk workgroups also publishes the chunk's total.  The
// offset of a workgroup is the sum of the totals of the chunks before its own
// plus the sum of the words of the workgroups before it in its chunk: all of
// them plain reads of words that their owners publish without waiting for
// anybody (a word) or after one such wait (a total).
//   word:  bit 31 published, bits 14..27 rows, bits 0..13 nnz
//   total: bit 63 published, bits 31..61 rows, bits 0..30 nnz
// Workgroups per chunk.  Vectors: a large chunk, so that few totals are read (their workgroups run
// nearly in step and a total is there early).  Matrices and tensors: a smaller one; their partitions
// take unequal time, the waiting wavefronts poll the words of their chunk, and hundreds of them on
// the same 2 KB of words are slower (chunks of 64, 128 and 256, us: two DCSR matrices of 20M 164, 159, 163; two CSR matrices of
// 10M doubles 118, 113, 114; three tensors of 4M doubles 119, 118, 119; three coordinate lists of 4M doubles 114, 110, 117; four
// and more operands are 1 % faster with 64, five DCSR matrices of 3M doubles 129, 131, 136).
// Products: smaller still, their partitions differ most (64 and 128, us: two CSR matrices of 10M 71.7, 75.3; three of 5M 78.6,
// 81.0; two DCSR matrices of 10M 102.0, 103.2; three coordinate lists of 5M 96.4, 97.5).
constexpr int kChunkVector = 512, kChunkOther = 128, kChunkProduct = 64;
constexpr int chunk_size(int fmt, bool mul) { return fmt == SPADD_VECTOR ? kChunkVector : (mul ? kChunkProduct : kChunkOther); }
constexpr int word_loads(int chunk) { return (chunk + NACHO_WAVE - 1) / NACHO_WAVE; }   // words of a chunk a lane reads
constexpr int kSpinLimit = 1 << 14;   // polls (each a sleep + one round trip to memory: tens of milliseconds in all)
constexpr unsigned kWordValid = 0x80000000u;
constexpr unsigned long long kTotalValid = 1ull << 63;
static_assert(kThreads * 11 < (1 << 14), "a partition's counts fit the 14-bit fields of its word");

__device__ inline unsigned long long pack_counts(long long rows, long long nnz)
{
    return ((unsigned long long)rows << 31) | (unsigned long long)nnz;
}


// Pointers into the operands' and the result's arrays are global-memory pointers (the loads and
// stores below then need no address-space check).
#define NACHO_GLOBAL __attribute__((address_space(1)))
template <typename U> __device__ inline const NACHO_GLOBAL U *global_ptr(unsigned long long a)
{
    return reinterpret_cast<const NACHO_GLOBAL U *>(a);
}
template <typename U> __device__ inline NACHO_GLOBAL U *global_out(U *p)
{
    return reinterpret_cast<NACHO_GLOBAL U *>(reinterpret_cast<uintptr_t>(p));
}

// ---- scans over the lanes of a wavefront with DPP moves (a shuffle goes through the LDS unit and takes
// ten times as long; these sit on the path every later workgroup waits for) --------------------------
template <int kCtrl, int kRowMask> __device__ inline int dpp_move(int identity, int v)
{
    return __builtin_amdgcn_update_dpp(identity, v, kCtrl, kRowMask, 0xf, false);
}
__device__ inline int dpp_scan_add(int v)              // inclusive
{
    v += dpp_move<0x111, 0xf>(0, v);                   // row_shr:1, 2, 4, 8: inside 16 lanes
    v += dpp_move<0x112, 0xf>(0, v);
    v += dpp_move<0x114, 0xf>(0, v);
    v += dpp_move<0x118, 0xf>(0, v);
    v += dpp_move<0x142, 0xa>(0, v);                   // row_bcast:15 into rows 1 and 3
    v += dpp_move<0x143, 0xc>(0, v);                   // row_bcast:31 into rows 2 and 3
    return v;
}
__device__ inline int dpp_scan_max(int v, int identity)
{
    v = max(v, dpp_move<0x111, 0xf>(identity, v));
    v = max(v, dpp_move<0x112, 0xf>(identity, v));
    v = max(v, dpp_move<0x114, 0xf>(identity, v));
    v = max(v, dpp_move<0x118, 0xf>(identity, v));
    v = max(v, dpp_move<0x142, 0xa>(identity, v));
    v = max(v, dpp_move<0x143, 0xc>(identity, v));
    return v;
}
__device__ inline int dpp_sum(int v) { return __builtin_amdgcn_readlane(dpp_scan_add(v), NACHO_WAVE - 1); }
__device__ inline int lane_before(int v, int first) { return dpp_move<0x138, 0xf>(first, v); }    // wave_shr:1
__device__ inline int lane_after(int v, int last) { return dpp_move<0x130, 0xf>(last, v); }       // wave_shl:1
__device__ inline unsigned long long lane_word(unsigned long long v, int from)
{
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, from);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(v >> 32), from);
    return ((unsigned long long)hi << 32) | lo;
}
// The value of the next lane (the last one: of b's first lane); of lane `from`.
__device__ inline int next_lane(int a, int b) { return lane_after(a, __builtin_amdgcn_readlane(b, 0)); }
__device__ inline float next_lane(float a, float b) { return __int_as_float(next_lane(__float_as_int(a), __float_as_int(b))); }
__device__ inline int lane_at(int v, int from) { return __builtin_amdgcn_ds_bpermute(from << 2, v); }
__device__ inline float lane_at(float v, int from) { return __int_as_float(lane_at(__float_as_int(v), from)); }
__device__ inline double lane_at(double v, int from)
{
    const long long x = __double_as_longlong(v);
    return __longlong_as_double((long long)lane_at((int)(x >> 32), from) << 32 | (unsigned)lane_at((int)(unsigned)x, from));
}
__device__ inline int lanes_below(unsigned long long mask)     // set bits of the mask below this lane
{
    return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
}
// Leading zeros of a word; none set: all ones (the instruction's own answer, for which the compiler would add a comparison and a choice).
__device__ inline uint32_t leading_zeros(uint32_t v)
{
    uint32_t n;
    asm("v_ffbh_u32 %0, %1" : "=v"(n) : "v"(v));
    return n;
}
// This lane's bit of a mask every lane agrees on.
__device__ inline bool my_bit(unsigned long long mask) { return __builtin_amdgcn_inverse_ballot_w64(mask); }

// Barrier of the workgroup for what its wavefronts exchange through LDS.  (__syncthreads also waits for every
// global load in flight; here those travel on.)
__device__ inline void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}


// LDS state of one partition.
template <typename KeyT, typename S, bool kRows, bool kRowHeads, bool kCsr, bool kSlices>
struct Tile {
    // The staged words: run t's entries from word sb[t] on, its sentinel behind them.  64-bit keys: the
    // columns are staged in the first half, the row ids of the row starts in the second, and the keys are
    // written over both.  (Tensors: the row field above its 32nd bit in `order`.)
    alignas(16) KeyT keys[S::kWords];
    // Order words by place: which staged word the place's entry is in (two operands: the byte offset of its
    // key; more: operand << 13 | word).  Before the keys are formed, with 32-bit keys: the row field of every
    // entry that starts a row.
    uint16_t order[S::kWords];
    unsigned long long starts[kRows ? S::kBlocks + 1 : 1];     // by staged word: a row starts here
    unsigned long long heads[S::kBlocks + 1];                  // by place: key differs from the one before
    unsigned long long row_heads[kRowHeads ? S::kBlocks + 1 : 1];      // ... its row (fibre) does
    unsigned long long slice_heads[kSlices ? S::kBlocks + 1 : 1];      // ... its slice does
    unsigned long long emitted[kCsr ? S::kBlocks : 1];         // CSR: the emitted places of a block
    int32_t block_before[kCsr ? S::kBlocks : 1];               // ... and how many its wavefront emits before it
    uint32_t wave_counts[kWaves], wave_slices[kWaves];         // emitted | row heads << 16; slice heads
    int32_t wave_before[kWaves];          // CSR: emitted by the wavefronts before
    uint16_t behind[kWaves][kMaxRuns];    // products: order words of the places behind a wavefront's last one
    unsigned long long sval[kMaxRuns];    // sums: address of the values of run t, biased: [staged word] is the entry's
    unsigned long long scol[kMaxRuns];    // remapped operands: the same for the columns
    unsigned long long srow[kMaxRuns];    // remapped operands: start[t]
    unsigned long long spos[kMaxRuns];    // remapped operands: pos of run t
    uint32_t cont, cont_next, cont_slice; // does the partition (the next one) start inside a row / slice
    uint32_t overflow;                    // the rows do not fit the key's row field
    int32_t base_nnz, base_rows, base_slices;      // output of the workgroups before this one in its chunk ...
    int32_t more_nnz, more_rows, more_slices;      // ... and of the chunks before
    int32_t gave_up;
};

template <int FMT, typename T, typename KeyT, int kSize>
using TileOf = Tile<KeyT, Shape<KeyT, T, kSize>, FMT != SPADD_VECTOR, FMT == SPADD_DCSR || FMT == SPADD_CSF3, FMT == SPADD_CSR,
                    FMT == SPADD_CSF3>;

// One thread's share of the stable merge of the sorted runs X = keys[sx, sx + nx)
// and Y = keys[sy, sy + ny) (nx, ny > 0), each followed by a sentinel key that no
// entry reaches: places d0 .. d0 + IPT - 1 of the merged order (X first on
// ties).  `steps` >= number of bits of min(nx, ny).  Places past nx + ny come
// out as garbage.  Reads only.  All positions are kept as byte offsets into the keys.
// emit(j, byte offset of the place's key, from X, the key, the key of the place before it or the
// sentinel when there is none).
template <typename KeyT, int IPT, class Emit>
__device__ __forceinline__ void merge_share(const char *kb, int sx, int nx, int sy, int ny, int d0, int steps, Emit &&emit)
{
    constexpr int KB = (int)sizeof(KeyT);
    // The diagonal: how many of the first d0 places come from X -- the search of Section 3.2 on two
    // one-level operands: the highest c in [lo, hi] such that X[c - 1] comes before Y[d0 - c]
    // (true for every c up to the answer, false beyond it), by binary lifting.
    const int lo = d0 - ny > 0 ? d0 - ny : 0, hi = d0 < nx ? d0 : nx;
    const int bx = (sx - 1) * KB;              // X[c - 1] lives at bx + c * KB: `at` for the c in hand
    const int by = (sy + d0) * KB + bx;        // Y[d0 - c] at by - at
    int at = bx + lo * KB;
    const int most = bx + hi * KB;
    // (four ways a step: half the dependent round trips to LDS)
    for (int step = KB << ((steps - 1) & ~1); step >= KB; step >>= 2) {
        KeyT xv[3], yv[3];
        int cand[3];
#pragma unroll
        for (int g = 0; g < 3; ++g) {
            cand[g] = at + (g + 1) * step;
            cand[g] = cand[g] < most ? cand[g] : most;
            xv[g] = *reinterpret_cast<const KeyT *>(kb + cand[g]);
            yv[g] = *reinterpret_cast<const KeyT *>(kb + (by - cand[g]));
        }
#pragma unroll
        for (int g = 0; g < 3; ++g) at = xv[g] <= yv[g] ? cand[g] : at;
    }
    int xi = at + KB, yi = by - at;
    // the keys in hand and the ones after them: a key is asked for two steps before it is compared
    KeyT xk = *reinterpret_cast<const KeyT *>(kb + xi), yk = *reinterpret_cast<const KeyT *>(kb + yi);
    KeyT xn = *reinterpret_cast<const KeyT *>(kb + xi + KB), yn = *reinterpret_cast<const KeyT *>(kb + yi + KB);
    // the key of the place before: the larger of the two last ones taken
    KeyT prev = ~KeyT(0);
    {
        const KeyT xp = *reinterpret_cast<const KeyT *>(kb + xi - KB), yp = *reinterpret_cast<const KeyT *>(kb + yi - KB);
        const bool hx = xi > sx * KB, hy = yi > sy * KB;
        if (hx) prev = xp;
        if (hy && (!hx || yp > xp)) prev = yp;
    }
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        const bool tx = xk <= yk;              // (an exhausted run shows its sentinel)
        const int src = tx ? xi : yi;
        const KeyT key = tx ? xk : yk;
        KeyT nk = 0;
        if (j + 2 < IPT) nk = *reinterpret_cast<const KeyT *>(kb + src + 2 * KB);
        emit(j, src, tx, key, prev);
        prev = key;
        const int next = src + KB;
        xi = tx ? next : xi;
        yi = tx ? yi : next;
        xk = tx ? xn : xk;
        yk = tx ? yk : yn;
        xn = tx ? nk : xn;
        yn = tx ? yn : nk;
    }
}

// Prefix look-up, first level: the 14-bit fields of the words of workgroups c0 .. c0 + m - 1 (m <= kChunk)
// summed over the wavefront, once every one of them is published.  `early` holds the words as they were
// when the wavefront asked for them ahead of time (kUseEarly), else the first round loads them too.
// Returns false when the wavefront gives up waiting.
template <bool kUseEarly, int kWordLoads>
__device__ inline bool sum_words(const unsigned int *words, int64_t c0, int m, const unsigned (&early)[kWordLoads],
                                 int lane, int &lo14, int &hi14)
{
    // (a word that has been seen published is not read again: a waiting wavefront only polls the words
    // it still misses -- hundreds of waiting workgroups re-reading whole chunks would load the fabric
    // that the publishing stores travel on)
    unsigned v[kWordLoads];
#pragma unroll
    for (int i = 0; i < kWordLoads; ++i) {
        const int j = i * NACHO_WAVE + lane;
        const bool mine = i * NACHO_WAVE < m && j < m;
        v[i] = mine ? 0u : kWordValid;
        if (kUseEarly && mine) v[i] = early[i];
    }
    for (int spins = 0;; ++spins) {
        bool missing = false;
#pragma unroll
        for (int i = 0; i < kWordLoads; ++i) {
            if (i * NACHO_WAVE < m && !(v[i] & kWordValid))
                v[i] = __hip_atomic_load(&words[c0 + i * NACHO_WAVE + lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            missing = missing || !(v[i] & kWordValid);
        }
        if (__ballot(missing) == 0ull) break;
        if (spins > kSpinLimit) return false;      // a predecessor has not published yet
        __builtin_amdgcn_s_sleep(16);
    }
    int l_lo = 0, l_hi = 0;
#pragma unroll
    for (int i = 0; i < kWordLoads; ++i) {
        l_lo += (int)(v[i] & 0x3fffu);
        l_hi += (int)((v[i] >> 14) & 0x3fffu);
    }
    lo14 = dpp_sum(l_lo);
    hi14 = dpp_sum(l_hi);
    return true;
}

// Second level: the two 31-bit fields of the totals of chunks 0 .. chunk - 1, summed, once published.
template <int kChunk>
__device__ inline bool sum_totals(const unsigned long long *totals, const unsigned int *words, int64_t chunk, int lane,
                                  unsigned long long early, int &lo31, int &hi31)
{
    // A total that its chunk's last workgroup has not published yet (that workgroup first has to get to
    // its own prefix sum) is not waited for: the words of that chunk are summed here -- they may all be
    // there long before, published early.
    int c_lo = 0, c_hi = 0;                        // (all entries together stay below 2^31)
    const unsigned none[word_loads(kChunk)] = {};
    for (int64_t first = 0; first < chunk; first += NACHO_WAVE) {
        const int64_t j = first + lane;
        unsigned long long s = j < chunk ? (first == 0 ? early : 0ull) : kTotalValid;
        if (s == 0ull) s = __hip_atomic_load(&totals[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const bool there = (s & kTotalValid) != 0;
        c_lo += dpp_sum(there ? (int)(s & 0x7fffffffull) : 0);
        c_hi += dpp_sum(there ? (int)((s >> 31) & 0x7fffffffull) : 0);
        unsigned long long missing = __ballot(!there);
        while (missing) {                          // (uniform)
            const int64_t jm = first + (__ffsll((long long)missing) - 1);
            missing &= missing - 1;
            int l = 0, h = 0;
            if (!sum_words<false, word_loads(kChunk)>(words, jm * kChunk, kChunk, none, lane, l, h)) return false;
            c_lo += l;
            c_hi += h;
        }
    }
    lo31 = c_lo;
    hi31 = c_hi;
    return true;
}

// Everything a launch passes, one kernel argument: the kernel reads the fields of it where it needs them
// (scalar loads from the argument segment) instead of holding them all from the start.
struct MergeArgs {
    DevOperands ops;
    SpaddValues vals;
    int64_t P, n_chunks;
    const int32_t *coord, *posn;
    unsigned long long *tile_state;
    SpaddOut out;
    MergeFields fields;
    WaveLog wlog;
    SpaddSearch search;
};
typedef const __attribute__((address_space(4))) MergeArgs *ArgPtr;

// kMul: the k-way intersection with products (an entry is emitted when all k
// operands store its coordinate, Section 2.1) instead of the union with sums;
// the partitions, the merge and the prefix sum are the same.
// kMapped: the operands are remapped ones (Section 3.3): CSR over the rows all
// operands store, positions counted over those rows only; the entries of row
// i' of operand t are read from start[t][i'] on.
// kSearch (sparse vectors): there is no partition kernel before this one; wavefronts 0 and 1 of the
// workgroup search its two boundaries themselves (Algorithm 1, equal-share queries) and store them in
// the partition table on the way -- the search fused into the executing kernel.
// A partition whose rows do not fit the row field of its keys is merged by searches (`far` below).
template <int FMT, typename T, typename KeyT, int kSize, int K, bool kMul, bool kMapped, bool kSearch>
__device__ __forceinline__ void merge_partition(ArgPtr arg_ptr, TileOf<FMT, T, KeyT, kSize> &w, const DevOperands &search_ops,
                                                const WaveStamp &stamp)
{
    static_assert(!kSearch || (FMT == SPADD_VECTOR && !kMapped), "the fused search is built for sparse vectors");
    // (the fields are read afresh after every call of this: left to itself the compiler reads all of them at the
    // start and spills what does not fit the scalar registers)
    auto fresh = [&]() { asm volatile("" : "+s"(arg_ptr)); };
    int64_t P = arg_ptr->P;
    if (kMapped && arg_ptr->ops.dyn_plan) {
        // the number of partitions is a result of earlier kernels of the call: the launch is sized for
        // an upper bound and the workgroups past the last partition have nothing to do
        P = arg_ptr->ops.dyn_plan[0];
        if ((int64_t)blockIdx.x >= P || arg_ptr->ops.dyn_plan[3]) return;      // (nor after an abandoned row loop)
    }
    typedef Shape<KeyT, T, kSize> S;
    constexpr int D = FMT == SPADD_VECTOR ? 1 : (FMT == SPADD_CSF3 ? 3 : 2);
    constexpr int kChunk = chunk_size(FMT, kMul), kWordLoads = word_loads(kChunk);
    constexpr bool kCsf = FMT == SPADD_CSF3;   // third-order tensors: three compressed levels
    constexpr bool kCoo = FMT == SPADD_COO;    // coordinate lists: the row of an entry is stored with it
    constexpr bool kWindow = D >= 2 && !kCoo;  // rows (fibres) come from pos arrays
    constexpr bool kRowHeads = FMT == SPADD_DCSR || kCsf;
    constexpr bool kWide = sizeof(KeyT) == 8;
    constexpr bool kDirect = !kMapped;         // the columns are copied to LDS by the memory pipeline
    constexpr int R = S::kIpt, NB = S::kBlocks;
    constexpr int NR = K <= 2 ? 2 : (K <= 4 ? 4 : 8);     // runs of the merge tree (a power of two)
    constexpr KeyT kSentinel = ~KeyT(0);
    constexpr uint16_t kPastKey = 0xffff;

    const int tid = threadIdx.x;
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(tid / NACHO_WAVE);
    // (launch_one.  Products and sums of CSR matrices know it: three CSR matrices of 5M entries in all 39.0 to 38.2 us; sums of vectors of four
    // doubles and of tensors would spill)
    const int k = K <= 4 && (kMul || (K > 2 && FMT == SPADD_CSR)) ? K : arg_ptr->ops.k;        // <= K
    const int p = (int)blockIdx.x;             // the partition of this workgroup, p < P
    KeyT *keys = w.keys;
    uint32_t *cols = reinterpret_cast<uint32_t *>(w.keys);                  // staged columns (32-bit keys: the keys)
    uint32_t *wide_rows = reinterpret_cast<uint32_t *>(w.keys) + S::kWords; // 64-bit keys: row fields of the row starts
    const int cb = arg_ptr->fields.cb, jb = arg_ptr->fields.jb, ahead = arg_ptr->fields.touch;
    const KeyT col_mask = (KeyT(1) << cb) - KeyT(1);
    const KeyT slice_mask = (KeyT(1) << (cb + jb)) - KeyT(1);
    typedef const NACHO_GLOBAL int32_t *Ints;
    auto ints = [](const int32_t *a) { return global_ptr<int32_t>((unsigned long long)(uintptr_t)a); };
    auto pos_of = [&](int t, int m) -> Ints { return ints(arg_ptr->ops.lvl[t][m].pos); };
    auto crd_of = [&](int t, int m) -> Ints { return ints(arg_ptr->ops.lvl[t][m].crd); };
    // (the table is constant to this kernel: scalar loads)
    typedef const __attribute__((address_space(4))) int32_t *Table;
    auto table_pos = [&](int b, int t, int m) -> int { return ((Table)(uintptr_t)arg_ptr->posn)[((int64_t)b * k + t) * D + m]; };
    auto table_coord = [&](int b, int m) -> int { return ((Table)(uintptr_t)arg_ptr->coord)[(int64_t)b * D + m]; };
    auto row_extent = [&]() -> int64_t {               // rows of the (remapped) operands
        return arg_ptr->ops.dyn_head ? (int64_t)arg_ptr->ops.dyn_head[0] : arg_ptr->ops.lvl[0][0].extent;
    };
    auto level_count = [&](int t, int m) -> int {      // segments of level m
        if (FMT == SPADD_CSR && m == 0) return kMapped ? (int)row_extent() : (int)arg_ptr->ops.lvl[t][0].extent;
        return (int)arg_ptr->ops.lvl[t][m].count;
    };

    // ---- the segments of this partition -------------------------------------
    // One operand per lane: lane t holds where the partition's entries of operand t start, how many there are, and
    // the segments of the level above (rows; fibres of a tensor) they lie in.
    // (the operands' arrays: asked for together with the table, two scalar round trips in all)
    Ints entry_crd[K], seg_pos[kWindow ? K : 1], seg_crd[kWindow ? K : 1];
#pragma unroll
    for (int t = 0; t < K; ++t) {
        entry_crd[t] = crd_of(t, D - 1);
        if constexpr (kWindow) {
            seg_pos[t] = pos_of(t, D - 1);
            seg_crd[t] = kMapped ? ints(arg_ptr->ops.start[t]) : crd_of(t, D - 2);
        }
    }
    int q_v = 0, len_v = 0, ilo_v = 0, ihi_v = 0;
    int up_lo_v = 0, up_hi_v = 0;              // tensors: the slices they lie in
    int next_seg_v = 0;                        // CSR: the segment (row) the next partition starts in
    auto put = [&](int v, int t, int x) { return lane == t ? x : v; };
    int row0 = 0;                              // keys count rows (slices) from here
    auto of = [](int v, int t) { return __builtin_amdgcn_readlane(v, t); };
    if constexpr (kSearch) {
        __shared__ int own_bounds[2][K];
        if (wave < 2) {                        // (whole wavefronts)
            int found[K];
            search_boundary<K, 0>(search_ops, 1, P, 0, nullptr, arg_ptr->search.total, arg_ptr->search.coord,
                                  arg_ptr->search.posn, arg_ptr->search.cost, p + wave, found);
            if (lane == 0) {
#pragma unroll
                for (int t = 0; t < K; ++t) own_bounds[wave][t] = found[t];
            }
        }
        __syncthreads();
        if (lane < k) {
            q_v = own_bounds[0][lane];
            len_v = own_bounds[1][lane] - q_v;
        }
    } else {
#pragma unroll
        for (int t = 0; t < K; ++t) {
            if (t >= k) break;
            const int q = table_pos(p, t, D - 1);
            q_v = put(q_v, t, q);
            len_v = put(len_v, t, table_pos(p + 1, t, D - 1) - q);
            if constexpr (kWindow) {
                const int most = level_count(t, D - 2), next = table_pos(p + 1, t, D - 2);
                ilo_v = put(ilo_v, t, table_pos(p, t, D - 2));
                ihi_v = put(ihi_v, t, row_behind(next, most));
                if (FMT == SPADD_CSR) next_seg_v = put(next_seg_v, t, next);
                if constexpr (kCsf) {
                    const int last = level_count(t, 0) - 1, up = table_pos(p + 1, t, 0);
                    up_lo_v = put(up_lo_v, t, table_pos(p, t, 0));
                    up_hi_v = put(up_hi_v, t, up < last ? up : last);
                }
            }
        }
        if (D >= 2) row0 = table_coord(p, 0);
    }
    // Tensors: the coordinates of the first and the last of these slices, the last one's first fibre, the fibres of the boundary's slice.
    // Asked for here, the round trips lie beside the entries' own; behind the staging one wavefront takes all of them, four in a row
    // per operand, while the others wait.  Only two operands in long partitions with 32-bit keys: elsewhere the entries wait for the scalar round
    // trip longer than that (two tensors of 16M entries in all 110.6 to 108.6 us, of 16M doubles 127.3 to 125.0, of 6.5M to 8M equal; but three of 5.2M 66.7
    // and 69.4, two of 2M, one round of middle partitions, 34.9 and 35.6, two of 50k, 64-bit keys, 24.9 and 25.9).
    constexpr bool kSlicesAhead = kCsf && kSize == MERGE_LONG && !kWide && K <= 2;
    int first_v = 0, last_v = 0, second_v = 0, fibre_v = 0, fibre_end_v = 0, begin_v = 0;
    constexpr int kSliceWords = kSlicesAhead ? K : 1;
    int first_s[kSliceWords], last_s[kSliceWords], second_s[kSliceWords], fibre_s[kSliceWords], fibre_end_s[kSliceWords];
    if constexpr (kSlicesAhead) {
#pragma unroll
        for (int t = 0; t < K; ++t) {
            // (an operand without slices: any words that are there)
            const bool some = t < k && level_count(t, 0) > 0;
            const int lo = some ? of(up_lo_v, t) : 0, hi = some ? of(up_hi_v, t) : 0, last = some ? level_count(t, 0) - 1 : 0;
            const Table crd0 = some ? (Table)(uintptr_t)arg_ptr->ops.lvl[t][0].crd : (Table)(uintptr_t)arg_ptr->coord;
            const Table pos1 = some ? (Table)(uintptr_t)arg_ptr->ops.lvl[t][1].pos : (Table)(uintptr_t)arg_ptr->coord;
            first_s[t] = crd0[lo < hi ? lo : hi];
            last_s[t] = crd0[hi];
            second_s[t] = pos1[hi];
            fibre_s[t] = pos1[lo < last ? lo : last];
            fibre_end_s[t] = pos1[(lo < last ? lo : last) + 1];
        }
    }
    // Only an operand that violates its preconditions (unsorted or repeated
    // coordinates) can overflow the staging buffer: such a partition contributes
    // nothing and the call reports INVALID_ARG, but the prefix sum goes on.
    int n = dpp_sum(len_v);                    // <= kCapacity by the host's choice of the partition count
    bool broken = __ballot(len_v < 0 || len_v > S::kCapacity) != 0ull || n > S::kCapacity;
    if (broken) n = len_v = 0;
    bool far = false;                          // (matrices and tensors) the rows do not fit the keys
    uint32_t logged_items = 0, logged_rows = 0;    // (instrumented build) places / row heads this wavefront walked

    // (sums of matrices and of two tensors: a workgroup goes before the others of its compute unit until its counts are published --
    // everybody behind it waits for the slowest one, nobody for its output: two DCSR matrices of 20M 159.6 to 153.9 us, two tensors of
    // 6.5M entries in all 77.5 to 76.7; three vectors, whose partitions are alike, 57.7 to 60.0, the product of two DCSR matrices 150.5 to 154.
    // More tensors keep a workgroup before its counts for so long that the others' output waits: three of 12M entries in all 113.2 us without,
    // 117.0 with it, four 116.8 and 124.7, eight 168.4 and 176.6; of 3.5M, one round, 50.9 and 49.7, 57.6 and 56.9, 73.0 and 72.2)
    constexpr bool kFirst = FMT != SPADD_VECTOR && !kMul && (!kCsf || K <= 2);
    if constexpr (kFirst) __builtin_amdgcn_s_setprio(2);
    // ---- 1. staging -----------------------------------------------------------
    // staged word of the operand's first entry (the copy of a run starts on a 16-byte boundary), words in all
    const int lead_v = kDirect ? (q_v & 3) : 0;
    const int run_v = lane < K ? (lead_v + len_v + 4) & ~3 : 0;    // (one for the sentinel)
    const int sb_v = 4 + dpp_scan_add(run_v) - run_v + lead_v;
    const int words = 4 + dpp_sum(run_v);
    const unsigned long long live_mask = __ballot(len_v > 0);
    const int live = __popcll(live_mask);      // runs with entries, one of them:
    const int live_t = live_mask ? __ffsll((long long)live_mask) - 1 : 0;
    if constexpr (kDirect) {
        // (global memory to LDS; every run's copy ends with its last entry: whole 16-byte pieces, then up to
        // three words)
        typedef __attribute__((address_space(3))) uint32_t lds_word;
#pragma unroll
        for (int t = 0; t < K; ++t) {
            const int len = of(len_v, t);
            if (len == 0) continue;
            const int q = of(q_v, t), lead = q & 3;
            const NACHO_GLOBAL uint32_t *src = reinterpret_cast<const NACHO_GLOBAL uint32_t *>(entry_crd[t] + (q - lead));
            lds_word *dst = (lds_word *)(cols + of(sb_v, t) - lead);
            const int pieces = (lead + len) >> 2, rest = (lead + len) & 3;
            // (the wavefront that starts on a run rotates with the run: short runs do not all land on wavefront 0)
            const int turn = (wave + kWaves - (t & (kWaves - 1))) & (kWaves - 1);
            for (int c = turn * NACHO_WAVE; c < pieces; c += kThreads)
                if (c + lane < pieces) __builtin_amdgcn_global_load_lds(src + (c + lane) * 4, dst + c * 4, 16, 0, 0);
            if (turn == 0 && lane < rest)
                __builtin_amdgcn_global_load_lds(src + pieces * 4 + lane, dst + pieces * 4, 4, 0, 0);
        }
    }
    // (rows of the first 512 segments of every run -- as a rule all of them -- are asked for together with
    // the entries: one round trip to memory; fibres of a tensor, which are many: of the first 1024 or 1536)
    constexpr int kAhead = !kCsf ? 1 : (kSize == MERGE_SHORT ? (K <= 2 ? 2 : 1) : (K <= 2 ? 3 : (K <= 4 ? 2 : 1)));
    int seg_a[kWindow ? K : 1][kAhead], seg_b[kWindow ? K : 1][kAhead], seg_id[kWindow ? K : 1][kAhead];
    // segment i of run t, counted from the partition's first: the positions of its entries and its row (CSF: j of the fibre; remapped
    // operands: where its entries are stored).  (The first one's address is the same in all lanes: the loads take an offset each.)
    auto load_segment = [&](int t, int i, int &a, int &b, int &id) {
        if constexpr (kWindow) {
            const Ints pos = seg_pos[t] + of(ilo_v, t), crd = seg_crd[t] + of(ilo_v, t);
            a = pos[(unsigned)i];
            b = pos[(unsigned)i + 1u];
            if constexpr (FMT != SPADD_CSR || kMapped) id = crd[(unsigned)i];
        }
    };
    if constexpr (kWindow) {
#pragma unroll
        for (int t = 0; t < K; ++t) {
            const int segments = of(ihi_v, t) - of(ilo_v, t);
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                seg_a[t][u] = seg_b[t][u] = seg_id[t][u] = 0;
                if (u * kThreads + tid < segments) load_segment(t, u * kThreads + tid, seg_a[t][u], seg_b[t][u], seg_id[t][u]);
            }
        }
    }
    if constexpr (kSlicesAhead) {
#pragma unroll
        for (int t = 0; t < K; ++t) {
            first_v = put(first_v, t, first_s[t]);
            last_v = put(last_v, t, last_s[t]);
            second_v = put(second_v, t, second_s[t]);
            fibre_v = put(fibre_v, t, fibre_s[t]);
            fibre_end_v = put(fibre_end_v, t, fibre_end_s[t]);
        }
        // (one wavefront: where the entries of the boundary's slice start)
        if (wave == 0) {
            Ints pos2 = seg_pos[0];
#pragma unroll
            for (int t = 1; t < K; ++t) pos2 = lane == t ? seg_pos[t] : pos2;
            if (ilo_v < ihi_v) begin_v = pos2[fibre_v];
        }
    }
    // The run of a staged word and the word's place in it; a word that holds no entry stands for the first entry
    // of the partition (valid = false).
    const int first_word = of(sb_v, live_t);
    auto run_of = [&](int &s, bool &valid) {
        int t = 0, first = of(sb_v, 0), len = of(len_v, 0);
#pragma unroll
        for (int u = 1; u < K; ++u)
            if (s >= of(sb_v, u)) { t = u; first = of(sb_v, u); len = of(len_v, u); }
        valid = (unsigned)(s - first) < (unsigned)len;
        s = valid ? s : first_word;
        return valid ? t : live_t;
    };
    const int word0 = wave * (R * NACHO_WAVE);     // a wavefront's staged words: word0 + j * 64 + lane, j < R
    // coordinate lists: the rows of the thread's words
    int coo_row[kCoo ? R : 1];
    if constexpr (kCoo) {
        Ints row_at[K];
#pragma unroll
        for (int t = 0; t < K; ++t) row_at[t] = crd_of(t, 0) + (of(q_v, t) - of(sb_v, t));
        if (n > 0) {
#pragma unroll
            for (int j = 0; j < R; ++j) {
                int at = word0 + j * NACHO_WAVE + lane;
                bool valid;
                const int t = run_of(at, valid);
                Ints row = row_at[0];
#pragma unroll
                for (int u = 1; u < K; ++u) row = t == u ? row_at[u] : row;
                coo_row[j] = row[at];
            }
        }
    }
    if constexpr (D >= 2)
        for (int i = tid; i < NB + 1; i += kThreads) w.starts[i] = 0ull;
    for (int i = tid; i < NB + 1; i += kThreads) {
        w.heads[i] = 0ull;
        if (kRowHeads) w.row_heads[i] = 0ull;
        if (kCsf) w.slice_heads[i] = 0ull;
    }
    if (wave == 0) {
        // addresses, biased so that a staged word indexes them
        unsigned long long val_v = 0ull, col_v = 0ull, row_v = 0ull, pos_v = 0ull;
        auto put2 = [&](unsigned long long v, int t, const void *base, int64_t bytes) {
            const unsigned long long x = (unsigned long long)(uintptr_t)base + (unsigned long long)bytes;
            return ((unsigned long long)(unsigned)put((int)(v >> 32), t, (int)(x >> 32)) << 32) |
                   (unsigned)put((int)(unsigned)v, t, (int)(unsigned)x);
        };
#pragma unroll
        for (int t = 0; t < K; ++t) {
            const int64_t bias = of(q_v, t) - of(sb_v, t);
            if constexpr (!kMul) val_v = put2(val_v, t, arg_ptr->vals.v[t], bias * (int64_t)sizeof(T));
            if (kMapped) {
                col_v = put2(col_v, t, arg_ptr->ops.lvl[t][1].crd, bias * 4);
                row_v = put2(row_v, t, arg_ptr->ops.start[t], 0);
                pos_v = put2(pos_v, t, arg_ptr->ops.lvl[t][1].pos, 0);
            }
        }
        if (lane < K) {
            if constexpr (!kMul) w.sval[lane] = val_v;
            if (kMapped) w.srow[lane] = row_v;
            if (kMapped) { w.scol[lane] = col_v; w.spos[lane] = pos_v; }
            // (the copies leave the word behind a run's last entry alone: its sentinel)
            if (kDirect) cols[sb_v + len_v] = ~0u;
        }
        if (lane == 0) {
            w.cont = w.cont_next = w.cont_slice = 0u;
            w.overflow = 0u;
            w.gave_up = 0;
        }
    }
    __syncthreads();                           // vectors: the keys are there; others: bits and flags are cleared
    unsigned long long st = 0ull;              // lane l: the starts of block wave * R + l
    int latest = 0;                            // latest row start before the block in hand (0: none yet)
    const uint32_t upto_lo = lane >= 31 ? ~0u : (2u << lane) - 1u;
    const uint32_t upto_hi = lane == 63 ? ~0u : (lane >= 32 ? (2u << (lane - 32)) - 1u : 0u);
    // the row start at or before word word0 + j * 64 + lane (called for j = 0, 1, ...)
    auto start_of = [&](int j) -> int {
        const unsigned long long x = lane_word(st, j);
        int e = latest;
        if (x) {                           // (uniform) some row starts in the block
            // how far it lies from the block's last word: the nearest of the start in the upper half, the lower half (32 more; none
            // stays the largest number) and the one before the block
            const uint32_t lo = (uint32_t)x & upto_lo, hi = (uint32_t)(x >> 32) & upto_hi;
            const int end = word0 + j * NACHO_WAVE + NACHO_WAVE - 1;
            const uint32_t from_hi = leading_zeros(hi), from_lo = leading_zeros(lo) | 32u;
            e = end - (int)min(min(from_hi, from_lo), (uint32_t)(end - latest));
            latest = end - __clzll((long long)x);
        }
        return e;
    };
    if constexpr (D >= 2) {
        if constexpr (kWindow) {
            auto mark_start = [&](int s, KeyT field) {
                atomicOr(reinterpret_cast<uint32_t *>(w.starts) + (s >> 5), 1u << (s & 31));
                if (kWide) wide_rows[s] = (uint32_t)field;
                if (!kWide) w.order[s] = (uint16_t)field;
                else if (kCsf) w.order[s] = (uint16_t)(field >> (kWide ? 32 : 0));
            };
            const uint32_t limit = arg_ptr->fields.limit;
#pragma unroll
            for (int t = 0; t < K; ++t) {
                const int i_lo = of(ilo_v, t), i_hi = of(ihi_v, t), q = of(q_v, t), len = of(len_v, t), sb = of(sb_v, t);
                int up_lo = 0, up_first = 0, up_last = 0, second_at = 0x7fffffff;  // tensors: the (at most two) slices
                bool many = false;
                if constexpr (kCsf) {
                    if (i_lo < i_hi) {
                        up_lo = of(up_lo_v, t);
                        const int up_hi = of(up_hi_v, t);
                        many = up_hi > up_lo + 1;
                        const Table crd0 = (Table)(uintptr_t)arg_ptr->ops.lvl[t][0].crd;       // (constant to this kernel)
                        up_first = kSlicesAhead ? of(first_v, t) : crd0[up_lo < up_hi ? up_lo : up_hi];
                        up_last = kSlicesAhead ? of(last_v, t) : crd0[up_hi];
                        if (up_hi == up_lo + 1)
                            second_at = kSlicesAhead ? of(second_v, t) : ((Table)(uintptr_t)arg_ptr->ops.lvl[t][1].pos)[up_hi];
                    }
                }
                if (t < k) {
                    // Does this partition (the next one) start inside a row, i.e. does some operand hold an
                    // entry of the boundary's row before the boundary?  Then that row's first output entry
                    // belongs to an earlier partition.  The boundary's row is the first (last) segment.
                    const int a0 = seg_a[t][0], id0 = seg_id[t][0];
                    if constexpr (kCsf) {
                        const int i0 = of(up_lo_v, t);
                        if (i_lo < i_hi && i0 < level_count(t, 0) && up_first == row0) {       // (uniform)
                            const Table pos1 = (Table)(uintptr_t)arg_ptr->ops.lvl[t][1].pos;
                            const int f1 = kSlicesAhead ? of(fibre_end_v, t) : pos1[i0 + 1];
                            const int f0 = kSlicesAhead ? 0 : pos1[i0], begin = kSlicesAhead ? of(begin_v, t) : 0;
                            if (tid == 0) {
                                if (i_lo < f1 && id0 == table_coord(p, 1) && q > a0) w.cont = 1u;
                                if (q > (kSlicesAhead ? begin : seg_pos[t][f0])) w.cont_slice = 1u;
                            }
                        }
                    } else if (tid == 0 && i_lo < i_hi && (FMT == SPADD_CSR || id0 == row0) && q > a0) w.cont = 1u;
                    if (FMT == SPADD_CSR) {
                        const int i_next = of(next_seg_v, t);
                        if (i_next < i_hi) {                       // (uniform)
                            if (i_next - i_lo < kThreads) { if (tid == i_next - i_lo && q + len > a0) w.cont_next = 1u; }
                            else if (tid == 0 && q + len > seg_pos[t][i_next]) w.cont_next = 1u;
                        }
                    }
                }
                if (len == 0) continue;
                constexpr int kMore = !kCsf && kSize != MERGE_SHORT && K <= 4 ? 8 : 4;      // segments a thread has in flight (registers)
                auto mark_segment = [&](int r, int a, int b, int id) {       // (segment i_lo + r)
                    const int s = a > q ? a : q;
                    if (b <= s || s >= q + len) return;            // nothing of it lies in the partition
                    uint32_t up;                                   // row, or slice of the fibre, counted from row0
                    KeyT field;
                    if constexpr (kCsf) {
                        up = (uint32_t)((r < second_at - i_lo ? up_first : up_last) - row0);
                        if (many) {                                // (uniform)
                            const int i = i_lo + r;
                            const Ints pos1 = pos_of(t, 1);
                            int lo = up_lo, hi = of(up_hi_v, t);
                            while (lo < hi) {                      // the last slice that starts at or before fibre i,
                                const int step = (hi - lo + 3) >> 2;       // four ways: half the dependent loads
                                int at[3], first[3];
#pragma unroll
                                for (int g = 0; g < 3; ++g) {
                                    at[g] = lo + (g + 1) * step < hi ? lo + (g + 1) * step : hi;
                                    first[g] = pos1[at[g]];
                                }
#pragma unroll
                                for (int g = 2; g >= 0; --g) hi = first[g] > i ? at[g] - 1 : hi;
#pragma unroll
                                for (int g = 0; g < 3; ++g) lo = first[g] <= i ? at[g] : lo;
                            }
                            up = (uint32_t)(crd_of(t, 0)[lo] - row0);
                        }
                        field = ((KeyT)up << jb) | (KeyT)(uint32_t)id;
                    } else {
                        up = FMT == SPADD_CSR ? (uint32_t)(r + (i_lo - row0)) : (uint32_t)(id - row0);
                        field = (KeyT)up;
                    }
                    const int at = s + (sb - q);
                    mark_start(at, field);
                    // (remapped operands: how far the row is stored from where it is counted; two of them: from its staged words)
                    if (kMapped) cols[at] = (uint32_t)(id - a + (K <= 2 ? q - sb : 0));
                    if (up >= limit) {
                        // past the key: the whole field over the column, and a mark that no other field has
                        w.overflow = 1u;
                        if (!kWide || kCsf) w.order[at] = kPastKey;
                        if (!kWide) cols[at] = (uint32_t)field;
                        else if (kCsf) { cols[at] = up; wide_rows[at] = (uint32_t)id; }
                    }
                };
#pragma unroll
                for (int u = 0; u < kAhead; ++u)
                    mark_segment(u * kThreads + tid, seg_a[t][u], seg_b[t][u], seg_id[t][u]);
                // (unsigned, as rows below: a segment behind the last one may lie past 2^31)
                const unsigned segments = (unsigned)(i_hi > i_lo ? i_hi - i_lo : 0);
                for (unsigned i = (unsigned)(tid + kAhead * kThreads); i < segments; i += kThreads * kMore) {
                    int a[kMore], b[kMore], id[kMore];
#pragma unroll
                    for (int u = 0; u < kMore; ++u) {
                        a[u] = b[u] = id[u] = 0;
                        if (i + u * kThreads < segments) load_segment(t, (int)(i + u * kThreads), a[u], b[u], id[u]);
                    }
#pragma unroll
                    for (int u = 0; u < kMore; ++u) mark_segment((int)(i + u * kThreads), a[u], b[u], id[u]);
                }
            }
            // the sentinel of a run: a row start whose row field is all ones, as its column is
            if (tid < K) mark_start(sb_v + len_v, kSentinel);
            __syncthreads();
            far = __builtin_amdgcn_readfirstlane((int)w.overflow) != 0 && !broken;
        }
        // Keys.  A wavefront takes R blocks of 64 words; the words' row starts are in its lanes, and where the
        // latest start before a block lies goes from block to block in a scalar register.
        if constexpr (kWindow) {
            if (lane < R) st = w.starts[wave * R + lane];
            int last = 0;
#pragma unroll
            for (int u = 0; u < (NB + NACHO_WAVE - 1) / NACHO_WAVE; ++u) {
                const int b = u * NACHO_WAVE + lane;
                const unsigned long long x = b < wave * R ? w.starts[b] : 0ull;
                if (x) last = b * 64 + 63 - __clzll((long long)x);
            }
            latest = __builtin_amdgcn_readlane(dpp_scan_max(last, 0), NACHO_WAVE - 1);
        }
        auto field_at = [&](int e) -> KeyT {
            if (!kWide) return (KeyT)w.order[e];
            return kCsf ? (KeyT)wide_rows[e] | (KeyT)w.order[e] << (kWide ? 32 : 0) : (KeyT)wide_rows[e];
        };
        if (kWindow && far) {
            // (the keys are put together in rank_far, where the code of such partitions lies together, out of the way of
            // the others': a small call waits for its instructions; the product of four CSR matrices of 10k entries 23.9 us with
            // it here, 23.1 there)
        } else if constexpr (!kWide && kWindow && kDirect) {
            // (all row fields are asked for, then put over the columns: block after block, each waits for a round trip to LDS.
            // What is written past the last word nobody reads)
            if (word0 < words) {                                   // (uniform)
                uint32_t f[R], c[R];
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    f[j] = (uint32_t)field_at(start_of(j));
                    c[j] = cols[word0 + j * NACHO_WAVE + lane];
                }
#pragma unroll
                for (int j = 0; j < R; ++j) cols[word0 + j * NACHO_WAVE + lane] = (f[j] << cb) | c[j];
            }
        } else {
            KeyT key[R];
            if constexpr (kCoo) {
                const uint32_t limit = arg_ptr->fields.limit;
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    int at = word0 + j * NACHO_WAVE + lane;
                    const uint32_t c = cols[at];
                    bool valid;
                    run_of(at, valid);
                    const uint32_t f = valid ? (uint32_t)(coo_row[j] - row0) : ~0u;
                    if (valid && f >= limit) w.overflow = 1u;
                    key[j] = ((KeyT)f << cb) | (KeyT)c;
                }
            } else {
                int e[R];
#pragma unroll
                for (int j = 0; j < R; ++j) e[j] = start_of(j);
#pragma unroll
                for (int j = 0; j < R; ++j) key[j] = field_at(e[j]) << cb;
                if constexpr (kMapped && K <= 2) {
                    // the words of the columns hold the rows' shifts so far.  A word without an entry asks for some column of its
                    // operand: its row field alone is past every entry's
                    const int second = of(sb_v, 1);
                    const Ints crd0 = crd_of(0, D - 1), crd1 = crd_of(K - 1, D - 1);
                    const unsigned last0 = (unsigned)arg_ptr->ops.lvl[0][D - 1].count - 1u, last1 = (unsigned)arg_ptr->ops.lvl[K - 1][D - 1].count - 1u;
                    uint32_t c[R];
#pragma unroll
                    for (int j = 0; j < R; ++j) {
                        const int at = word0 + j * NACHO_WAVE + lane;
                        const unsigned to = (unsigned)(at + (int)cols[e[j]]);
                        const Ints crd = at >= second ? crd1 : crd0;
                        c[j] = (uint32_t)crd[min(to, at >= second ? last1 : last0)];
                    }
#pragma unroll
                    for (int j = 0; j < R; ++j) key[j] |= (KeyT)c[j];
                } else if constexpr (kMapped) {
                    // the words of the columns hold the rows' shifts so far
                    uint32_t c[R];
#pragma unroll
                    for (int j = 0; j < R; ++j) {
                        int at = word0 + j * NACHO_WAVE + lane;
                        int sh = (int)cols[e[j]];
                        bool valid;
                        const int t = run_of(at, valid);
                        // (a word without an entry: the partition's first one, in its own row)
                        sh = valid ? sh : (n > 0 ? (int)cols[first_word] : 0);
                        c[j] = ~0u;
                        if (n > 0) c[j] = (uint32_t)global_ptr<int32_t>(w.scol[t])[at + sh];
                        c[j] = valid ? c[j] : ~0u;
                    }
#pragma unroll
                    for (int j = 0; j < R; ++j) key[j] |= (KeyT)c[j];
                } else {
#pragma unroll
                    for (int j = 0; j < R; ++j) key[j] |= (KeyT)cols[word0 + j * NACHO_WAVE + lane];
                }
            }
            if (kWide || kMapped) lds_barrier();       // (the keys go over the columns, row fields and shifts)
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const int s = word0 + j * NACHO_WAVE + lane;
                if (s < words) keys[s] = key[j];
            }
        }
        __syncthreads();
        if constexpr (kCoo) far = __builtin_amdgcn_readfirstlane((int)w.overflow) != 0 && !broken;
    }

    // ---- 1b. rows too far apart for the keys ------------------------------------------
    // The keys of such a partition are its row fields, which one word holds for any rows, slices and fibres (merge_fields), and
    // below them as many of the column's upper bits as there is room for.  Every entry searches its place in the other
    // operands' runs: a binary search in LDS and, only among words that equal its own, one in the operand's columns.
    // (Merging pairs of words would take a second word per entry, for which there is no LDS.  Searching rows and columns in
    // the operands' own arrays was bound by the gathers a compute unit's L1 takes, searching the columns of a long row by
    // their latency, unrolled searches by fetching their instructions, which no other partition of the XCD has run: two
    // matrices of 2M entries, eight of their 718 partitions far: 130, 98, 85 and, like this, 67 us a call.)  Values and
    // output go the way of every partition, but for the columns, which are stored once more in full.  The layout of the
    // keys is chosen so that few partitions come here.
    int row_at = cb;                           // the row field of a key starts at this bit
    if (__builtin_expect(far, 0)) {
        const int last = (int)row_extent() - 1, next = table_coord(p + 1, 0);
        const uint32_t most = (uint32_t)((next < last ? next : last) - row0);
        const int room = 8 * (int)sizeof(KeyT) - jb - (most > 0u ? 32 - __builtin_clz(most) : 0);
        row_at = room < 0 ? 0 : (room < cb ? room : cb);
    }
    auto row_field = [&](KeyT key) -> KeyT { return key >> row_at; };
    // (remapped operands) how far an entry of operand t is stored from where it is counted
    auto shift_of = [&](int t, KeyT field) -> int {
        if constexpr (!kMapped) return 0;
        const int row = row0 + (int)(uint32_t)field;
        return global_ptr<int32_t>(w.srow[t])[row] - global_ptr<int32_t>(w.spos[t])[row];
    };
    auto column_at = [&](int t, int s, KeyT field) -> int {
        if constexpr (kMapped) return global_ptr<int32_t>(w.scol[t])[s + shift_of(t, field)];
        int c = 0;
#pragma unroll 1
        for (int u = 0; u < k; ++u)
            if (t == u) c = crd_of(u, D - 1)[of(q_v, u) + (s - of(sb_v, u))];
        return c;
    };
    constexpr int KB = (int)sizeof(KeyT);
    const int place0 = wave * (R * NACHO_WAVE);    // a wavefront's places: place0 + j * 64 + lane, j < R
    const int block0 = wave * R;
    const unsigned two_at = K <= 2 ? (unsigned)(of(sb_v, K - 1) * KB) : 0u;    // two operands: the second one's words start here
    auto word_of = [&](unsigned o, int &t) -> int {    // the staged word an order word names, and its operand
        t = K <= 2 ? (K == 2 && o >= two_at ? 1 : 0) : (int)(o >> 13);
        return K <= 2 ? (int)(o / KB) : (int)(o & 0x1fffu);
    };
    auto rank_far = [&]() {
        if constexpr (D >= 2) {
            if constexpr (kWindow) {
                // the row fields
                if constexpr (!kWide) {
#pragma unroll 1
                    for (int j = 0; j < R && word0 + j * NACHO_WAVE < words; ++j) {
                        const int e = start_of(j);         // (a row start gets the field it holds)
                        cols[word0 + j * NACHO_WAVE + lane] = w.order[e] == kPastKey ? cols[e] : w.order[e];
                    }
                } else {
                    KeyT field[R];
#pragma unroll
                    for (int j = 0; j < R; ++j) {
                        const int e = start_of(j);
                        field[j] = (KeyT)wide_rows[e];
                        if (kCsf) field[j] |= w.order[e] == kPastKey ? (KeyT)cols[e] << jb : (KeyT)w.order[e] << (kWide ? 32 : 0);
                    }
                    lds_barrier();
#pragma unroll
                    for (int j = 0; j < R; ++j) {
                        const int s = word0 + j * NACHO_WAVE + lane;
                        if (s < words) keys[s] = field[j];
                    }
                }
                __syncthreads();
            }
#pragma unroll 1
            for (int u = 0; u < k; ++u) {
                const int q = of(q_v, u), sb = of(sb_v, u), len = of(len_v, u);
#pragma unroll 4
                for (int i = tid; i < len; i += kThreads) {
                    KeyT field;
                    if constexpr (kCoo) field = (KeyT)(uint32_t)(crd_of(u, 0)[q + i] - row0);
                    else field = keys[sb + i];
                    const uint32_t col = (uint32_t)crd_of(u, D - 1)[q + i + shift_of(u, field)];
                    keys[sb + i] = (field << row_at) | (KeyT)(row_at > 0 ? col >> (cb - row_at) : 0u);
                }
            }
            // (unsorted or repeated coordinates can give two entries one place and another place none: every order
            // word names an entry before the searches write theirs)
            for (int m = tid; m < n; m += kThreads)
                w.order[m] = (uint16_t)(K <= 2 ? first_word * (int)sizeof(KeyT) : (live_t << 13 | first_word));
            __syncthreads();
#pragma unroll 1
            for (int j = 0; j < R && word0 + j * NACHO_WAVE < words; ++j) {
                int s = word0 + j * NACHO_WAVE + lane;
                bool valid;
                const int t = run_of(s, valid);
                const KeyT key = keys[s];
                int place = 0;
                bool head = true;
#pragma unroll 1
                for (int u = 0; u < k; ++u) {
                    const int first = of(sb_v, u), end = first + of(len_v, u);
                    int at = s;                                    // the entries of u before this one: those in front of word `at`
                    if (t != u && first < end) {
                        at = first;
                        // (four ways a step, as in merge_share)
                        for (int step = 1 << ((31 - __builtin_clz((unsigned)(end - first))) & ~1); step > 0; step >>= 2) {
                            KeyT x[3];
                            int to[3];
#pragma unroll
                            for (int g = 0; g < 3; ++g) {
                                to[g] = at + (g + 1) * step < end ? at + (g + 1) * step : end;
                                x[g] = keys[to[g] - 1];
                            }
#pragma unroll
                            for (int g = 0; g < 3; ++g) at = x[g] < key ? to[g] : at;
                        }
                        if (at < end && keys[at] == key) {
                            // words that equal this one, as a rule one or two: steps that double, then halve
                            const KeyT field = row_field(key);
                            const int col = column_at(t, s, field);
                            const Ints cols_u = crd_of(u, D - 1) + (of(q_v, u) - first + shift_of(u, field));
                            bool up = true;
                            for (int step = 1; step > 0;) {
                                const int to = at + step;
                                const bool before = to <= end && keys[to - 1] == key && cols_u[to - 1] < col;
                                at = before ? to : at;
                                up = up && before;
                                step = up ? 2 * step : step >> 1;
                            }
                            if (u < t && at < end && keys[at] == key && cols_u[at] == col) { head = false; ++at; }
                        }
                    }
                    place += at - first;
                }
                if (valid) {
                    w.order[place] = (uint16_t)(K <= 2 ? s * (int)sizeof(KeyT) : (t << 13 | s));
                    // (few: the bits of the others are set below)
                    if (!head) atomicOr(reinterpret_cast<uint32_t *>(w.heads) + (place >> 5), 1u << (place & 31));
                }
            }
            __syncthreads();
            if constexpr (kRowHeads) {
                // rows and slices start where the fields of neighbours differ
#pragma unroll 1
                for (int j = 0; j < R && place0 + j * NACHO_WAVE < n; ++j) {
                    const int m = place0 + j * NACHO_WAVE + lane, mm = m < n ? m : n - 1;
                    int t;
                    const KeyT field = row_field(keys[word_of(w.order[mm], t)]), before = row_field(keys[word_of(w.order[mm > 0 ? mm - 1 : 0], t)]);
                    const unsigned long long in = low_bits(n - (place0 + j * NACHO_WAVE));
                    const unsigned long long rm = __ballot(m == 0 || field != before) & in;
                    const unsigned long long sm = __ballot(m == 0 || field >> jb != before >> jb) & in;
                    if (lane == 0) {
                        w.row_heads[block0 + j] = rm;
                        if (kCsf) w.slice_heads[block0 + j] = sm;
                    }
                }
            }
            if (lane < R) w.heads[block0 + lane] = ~w.heads[block0 + lane];
        }
    };

    // Sums of two and three coordinate lists and tensors (where merge_fields says so): a word of every line of the values is asked for beside the
    // merge, so that the lines are on their way from memory before the places ask for them.
    constexpr bool kTouch = !kMul && (kCoo || kCsf) && K <= 3;
    int touched[kTouch ? K : 1];
    if constexpr (kTouch) {
#pragma unroll
        for (int t = 0; t < K; ++t) touched[t] = 0;
        if (ahead) {                           // (uniform)
            int from = 0;                      // (the threads are shared out over the operands' lines)
#pragma unroll
            for (int t = 0; t < K; ++t) {
                const int len = of(len_v, t);
                if (len == 0) continue;
                constexpr int kLine = 128 / (int)sizeof(T);
                const int q = of(q_v, t), lines = (int)((unsigned)(q + len - 1) / kLine - (unsigned)q / kLine) + 1;
                int i = tid - from;
                i += i < 0 ? kThreads : 0;
                const int at = i * kLine < len ? i * kLine : len - 1;
                const auto values = global_ptr<T>((unsigned long long)(uintptr_t)arg_ptr->vals.v[t]) + q;
                if (i < lines) touched[t] = reinterpret_cast<const NACHO_GLOBAL int *>(values)[at * (int)(sizeof(T) / 4)];
                from = (from + lines) & (kThreads - 1);
            }
        }
    }

    // ---- 2. merge: adjacent runs pairwise, in rounds ------------------------------
    // (all of this is uniform over the workgroup except the thread's own share)
    const char *kb = reinterpret_cast<const char *>(w.keys);
    int mb = 0;                                // K > 2 or one run: the key of place m is keys[mb + m]
    bool moved = false;                        // the order words are in w.order (K > 2: from word mb on)
    bool marked = false;                       // the head bits are in place
    int only = live_t;                         // one run: its operand
    // sets the bits of the places d0 .. d0 + R - 1 (bit R - 1 - j: place d0 + j)
    auto set_bits = [&](int d0, uint32_t hm, uint32_t rm, uint32_t sm) {
        const int left = n - d0;
        const uint32_t in = left >= R ? (1u << R) - 1u : (1u << (left > 0 ? left : 0)) - 1u;
        auto put_bits = [&](unsigned long long *at, uint32_t m) {
            m = (__builtin_bitreverse32(m) >> (32 - R)) & in;
            uint32_t *a = reinterpret_cast<uint32_t *>(at) + (d0 >> 5);
            const int shift = d0 & 31;
            atomicOr(a, m << shift);
            if (shift + R > 32) atomicOr(a + 1, m >> (32 - shift));
        };
        put_bits(w.heads, hm);
        if constexpr (kRowHeads) put_bits(w.row_heads, rm);
        if constexpr (kCsf) put_bits(w.slice_heads, sm);
    };
    auto compare = [&](KeyT key, KeyT prev, uint32_t &hm, uint32_t &rm, uint32_t &sm) {
        // (comparison and addition with carry in inline assembly takes an instruction less a bit, but ties them to places between the others:
        // two vectors of 10M 77.9 to 80.8 us)
        if constexpr (!kRowHeads) hm += hm + (key != prev ? 1u : 0u);
        else {
            const KeyT diff = key ^ prev;
            hm += hm + (diff != 0 ? 1u : 0u);
            rm += rm + (diff > col_mask ? 1u : 0u);
            if (kCsf) sm += sm + (diff > slice_mask ? 1u : 0u);
        }
    };
    if (__builtin_expect(far, 0)) {
        rank_far();
        moved = marked = true;
    } else if constexpr (K <= 2) {
        if (live == 2) {
            const int nx = of(len_v, 0), ny = of(len_v, K - 1);
            const int d0 = tid * R;
            if (d0 < n) {
                const int steps = 32 - __builtin_clz((unsigned)(nx < ny ? nx : ny));
                uint32_t hm = 0, rm = 0, sm = 0;
                uint16_t *order = w.order + d0;
                merge_share<KeyT, R>(kb, of(sb_v, 0), nx, of(sb_v, K - 1), ny, d0, steps,
                                     [&](int j, int src, bool, KeyT key, KeyT prev) {
                    compare(key, prev, hm, rm, sm);
                    order[j] = (uint16_t)src;
                });
                set_bits(d0, hm, rm, sm);
            }
            moved = marked = true;
        } else if (live == 1) mb = of(sb_v, only);
    } else {
        int rs[NR], rn[NR], ro[NR];            // start and length of the runs still to be merged; operand, or -1: merged
        if (K == 3) {
            // three operands: the lone run is the one that makes the first round the shorter one
            const bool front = of(len_v, 2) < of(len_v, 0);         // (-, a), (b, c)  rather than  (a, b), (c, -)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int t = front ? g - 1 : g;
                rs[g] = 4;
                rn[g] = 0;
                ro[g] = 0;
#pragma unroll
                for (int u = 0; u < 3; ++u)
                    if (u == t) { rs[g] = of(sb_v, u); rn[g] = of(len_v, u); ro[g] = u; }
            }
        } else {
#pragma unroll
            for (int g = 0; g < NR; ++g) {
                rs[g] = g < K ? of(sb_v, g) : 4;
                rn[g] = g < K ? of(len_v, g) : 0;
                ro[g] = g;
            }
        }
#pragma unroll
        for (int s = 1; s < NR; s <<= 1) {
            const bool final_round = 2 * s == NR;
            int t_base = 0, steps = 0;
            int msx = 4, mnx = 0, msy = 4, mny = 0, md0 = -1, mox = 0, moy = 0;
            const bool carried = s > 1;        // (the entries' order words are in place; before, a staged word names itself)
#pragma unroll
            for (int g = 0; g < NR; g += 2 * s) {
                const int nx = rn[g], ny = rn[g + s];
                if (nx > 0 && ny > 0) {
                    const int tg = (nx + ny + R - 1) / R;              // threads of this pair
                    const int lesser = nx < ny ? nx : ny;
                    const int bits = 32 - __builtin_clz((unsigned)lesser);
                    steps = bits > steps ? bits : steps;
                    if (tid >= t_base && tid < t_base + tg) {
                        msx = rs[g]; mnx = nx; msy = rs[g + s]; mny = ny;
                        md0 = (tid - t_base) * R;
                        mox = carried ? 0 : ro[g] << 13;
                        moy = carried ? 0 : ro[g + s] << 13;
                    }
                    t_base += tg;
                } else if (!carried && live > 1) {
                    // a run without a partner in the first round: its order words, so that every later round finds them in place
                    const int first = nx > 0 ? rs[g] : rs[g + s], own = (nx > 0 ? ro[g] : ro[g + s]) << 13;
                    for (int i = first + tid; i < first + nx + ny; i += kThreads) w.order[i] = (uint16_t)(own | i);
                }
            }
            if (t_base > 0) {                  // (uniform) some pair has two non-empty sides
                KeyT mk[R];
                uint32_t mo[(R + 1) / 2];
                uint32_t hm = 0, rm = 0, sm = 0;
                if (md0 >= 0)
                    merge_share<KeyT, R>(kb, msx, mnx, msy, mny, md0, steps,
                                         [&](int j, int src, bool tx, KeyT key, KeyT prev) {
                        mk[j] = key;
                        const uint32_t at = (uint32_t)src / KB;
                        const uint32_t o = carried ? (uint32_t)w.order[at] : ((uint32_t)(tx ? mox : moy) | at);
                        mo[j / 2] = j & 1 ? mo[j / 2] | o << 16 : o;
                        if (final_round) compare(key, prev, hm, rm, sm);
                    });
                lds_barrier();                 // every share is read: the merged runs may overwrite their sources
                if (md0 >= 0) {
                    // (last round: what lies behind the last place is nobody's any more)
                    const int left = final_round ? R : mnx + mny - md0;
#pragma unroll
                    for (int j = 0; j < R; ++j)
                        if (j < left) {
                            keys[msx + md0 + j] = mk[j];
                            w.order[msx + md0 + j] = (uint16_t)(mo[j / 2] >> (16 * (j & 1)));
                        }
                    if (!final_round && md0 == 0) keys[msx + mnx + mny] = kSentinel;
                    if (final_round) set_bits(md0, hm, rm, sm);
                }
                if (final_round) marked = true;
                else lds_barrier();
            } else if (!carried && live > 1) lds_barrier();        // (the order words just written)
#pragma unroll
            for (int g = 0; g < NR; g += 2 * s) {
                if (rn[g] == 0) { rs[g] = rs[g + s]; ro[g] = ro[g + s]; }
                if (live > 1) ro[g] = -1;
                rn[g] += rn[g + s];
            }
        }
        mb = rs[0];
        moved = ro[0] < 0;
        only = ro[0];
    }
    // A partition that one run is left of before the last round, or from the start: the keys are in place
    // order, the bits come from comparing neighbours.
    const bool all_heads = !moved && !kRowHeads;       // (one operand: every place is a head)
    if (!marked && !all_heads) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int m = place0 + j * NACHO_WAVE + lane;
            if (place0 + j * NACHO_WAVE >= n) break;   // (uniform)
            const KeyT k0 = keys[mb + (m < n ? m : 0)], kp = keys[mb + (m < n ? m : 0) - 1];
            const KeyT diff = k0 ^ kp;
            const unsigned long long hm = __ballot(m < n && (m == 0 || diff != 0));
            if (lane == 0) w.heads[block0 + j] = hm;
            if constexpr (kRowHeads) {
                const unsigned long long rm = __ballot(m < n && (m == 0 || diff > col_mask));
                if (lane == 0) w.row_heads[block0 + j] = rm;
            }
            if constexpr (kCsf) {
                const unsigned long long sm = __ballot(m < n && (m == 0 || diff > slice_mask));
                if (lane == 0) w.slice_heads[block0 + j] = sm;
            }
        }
    }
    wave_sync();                               // (a wavefront's places are merged and marked by its own threads)

    // ---- the values: where an entry's is ---------------------------------------------------------
    // Products emit one place in k at most.  (launches for five and more operands: K = 8)
    constexpr int kLeast = K <= 4 ? K : 5, NP = (R + kLeast - 1) / kLeast;     // (a wavefront's emitted places, in 64s)
    T val[kMul ? NP : R], tail = T(0);
    // the value of the entry an order word names (byte offsets throughout: with two operands and values as long as the
    // keys the order word is the offset)
    auto value_at = [&](unsigned o) -> T {
        const unsigned t8 = K <= 2 ? (K == 2 && o >= two_at ? 8u : 0u) : (o >> 13) * 8u;
        const unsigned long long base = *reinterpret_cast<const unsigned long long *>(reinterpret_cast<const char *>(w.sval) + t8);
        const unsigned long long off = K <= 2 ? (unsigned long long)o * sizeof(T) / KB : (unsigned long long)(o & 0x1fffu) * sizeof(T);
        return *global_ptr<T>(base + off);
    };
    auto order_of = [&](int m) -> unsigned {
        if constexpr (K <= 2) return moved ? (unsigned)w.order[m] : (unsigned)((mb + m) * KB);
        else return moved ? (unsigned)w.order[mb + m] : (unsigned)(only << 13 | (mb + m));
    };
    // the order words of the wavefront's places (past the last place: any words)
    auto orders = [&](unsigned (&o)[R]) {
        const int m = place0 + lane;
        if (moved) {
            const uint16_t *order = w.order + (K <= 2 ? 0 : mb) + m;
#pragma unroll
            for (int j = 0; j < R; ++j) o[j] = order[j * NACHO_WAVE];
        } else {
            const unsigned first = K <= 2 ? (unsigned)((mb + m) * KB) : (unsigned)(only << 13 | (mb + m));
#pragma unroll
            for (int j = 0; j < R; ++j) o[j] = first + (unsigned)(j * NACHO_WAVE * (K <= 2 ? KB : 1));
        }
    };

    // ---- 3. assembly: which places are emitted, and how many before every block -----------
    // lane l: block block0 + l of the wavefront's own (and, l = R, the one behind them)
    auto valid_bits = [&](int b) -> unsigned long long {
        return low_bits(n - b * NACHO_WAVE);
    };
    auto shifted = [](unsigned long long own, unsigned long long next, int g) {
        return (own >> g) | (next << (64 - g));        // 1 <= g <= 7
    };
    const unsigned long long in = lane <= R ? valid_bits(block0 + lane) : 0ull;
    unsigned long long e = in, r = 0ull, sl = 0ull, eq = 0ull, eq_next = 0ull;
    auto load_heads = [&]() {
        if (!all_heads && lane <= R) e = w.heads[block0 + lane] & in;
        // places whose key equals the one before
        eq = in & ~e;
        eq_next = ((unsigned long long)(unsigned)lane_after((int)(eq >> 32), 0) << 32) | (unsigned)lane_after((int)(unsigned)eq, 0);
    };
    // products: the order words of the wavefront's places and of those behind them
    unsigned product_words[kMul ? R : 1], word_behind = 0u;
    bool emits = false;                        // (uniform) the wavefront has something to emit
    if constexpr (kMul) {
        lds_barrier();                         // (whether the wavefront's last places are emitted hangs on the next ones)
        load_heads();
#pragma unroll
        for (int g = 1; g < K; ++g)
            if (g < k) e &= shifted(eq, eq_next, g);
        if (live < k || lane >= R) e = 0ull;
        emits = __ballot(e != 0ull) != 0ull;
        if (emits) {                           // (all operands have entries here, so the order words are in w.order)
            orders(product_words);
            word_behind = order_of(place0 + R * NACHO_WAVE + (lane < K ? lane : 0));
        }
    } else if (!all_heads && lane < R) e = w.heads[block0 + lane] & in;
    if constexpr (kRowHeads) {
        if (lane < R) r = w.row_heads[block0 + lane] & in;
        if (tid == 0 && w.cont) r &= ~1ull;          // the first row's head is elsewhere
    }
    if constexpr (kCsf) {
        if (lane < R) sl = w.slice_heads[block0 + lane] & in;
        if (tid == 0 && w.cont_slice) sl &= ~1ull;
    }
    const int block_counts = lane < R ? __popcll(e) | __popcll(r) << 16 : 0;
    const int wave_incl = dpp_scan_add(block_counts);
    int slice_incl = 0;
    if (lane == NACHO_WAVE - 1) w.wave_counts[wave] = (uint32_t)wave_incl;
    if constexpr (kCsf) {
        slice_incl = dpp_scan_add(lane < R ? __popcll(sl) : 0);
        if (lane == NACHO_WAVE - 1) w.wave_slices[wave] = (uint32_t)slice_incl;
    }
    if (FMT == SPADD_CSR && lane < R) {        // (read by all wavefronts after the prefix sum)
        w.emitted[block0 + lane] = e;
        w.block_before[block0 + lane] = wave_incl - block_counts;
    }
    lds_barrier();
    int own_counts = 0, wave_before = 0, own_slices = 0, slices_before = 0;
    {
        const int v = lane < kWaves ? (int)w.wave_counts[lane] : 0;
        const int incl = dpp_scan_add(v);
        own_counts = of(incl, kWaves - 1);
        wave_before = of(incl - v, wave);
        if (FMT == SPADD_CSR && tid < kWaves) w.wave_before[tid] = incl - v;
        if constexpr (kCsf) {
            const int v2 = lane < kWaves ? (int)w.wave_slices[lane] : 0;
            const int incl2 = dpp_scan_add(v2);
            own_slices = of(incl2, kWaves - 1);
            slices_before = of(incl2 - v2, wave);
        }
    }
    const int own_nnz = own_counts & 0xffff, own_rows = own_counts >> 16;

    // ---- 4. prefix sum over the workgroups, first half: publish -------------------------
    // state of the call: one total per chunk, one 32-bit word per workgroup; third-order tensors keep
    // a second such pair behind the first for the slices
    fresh();
    const int64_t n_chunks = arg_ptr->n_chunks, state_half = n_chunks + (P + 1) / 2;
    unsigned long long *totals = arg_ptr->tile_state;
    unsigned int *counts_of = reinterpret_cast<unsigned int *>(totals + n_chunks);
    unsigned long long *totals2 = totals + state_half;
    unsigned int *counts_of2 = reinterpret_cast<unsigned int *>(totals + state_half + n_chunks);
    const int64_t chunk = p / kChunk, chunk0 = chunk * kChunk;
    unsigned early[kWordLoads];
    if (wave == 0) {
        if (lane == 0) {
            __hip_atomic_store(&counts_of[p], kWordValid | ((unsigned)own_rows << 14) | (unsigned)own_nnz, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
            if (kCsf)
                __hip_atomic_store(&counts_of2[p], kWordValid | (unsigned)own_slices, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        }
    }

    if constexpr (kFirst) __builtin_amdgcn_s_setprio(0);
    // sums: every place asks for its value, straight from the operands (64 places read one contiguous stretch per operand).
    // Not before the counts are published: asking takes one to ten microseconds where the memory pipeline is full, and everybody
    // behind this workgroup waits for them (three vectors, 11M entries: 71.0 to 68.6 us; two DCSR matrices of 20M: 175 to 168).
    KeyT key[kMul ? NP : R];
    if constexpr (kTouch)
        if (ahead) {                           // (uniform; a call that asks for nothing does not wait here either)
#pragma unroll
            for (int t = 0; t < K; ++t) asm volatile("" ::"v"(touched[t]));    // (nobody's words, but the loads have to stay)
        }
    if constexpr (!kMul) if (n > 0) {
        unsigned o[R];
        orders(o);
        if (place0 + R * NACHO_WAVE > n) {         // (uniform: the wavefronts at the end)
            // past the last place: the first entry of an operand (with the last place's own entry three vectors take 62.1 us
            // instead of 61.5, two of 300k entries 11.1 instead of 10.3)
            const unsigned some = K <= 2 ? (unsigned)(of(sb_v, live_t) * KB) : (unsigned)(live_t << 13 | of(sb_v, live_t));
#pragma unroll
            for (int j = 0; j < R; ++j)
                if (place0 + j * NACHO_WAVE + lane >= n) o[j] = some;
        }
#pragma unroll
        for (int j = 0; j < R; ++j) val[j] = value_at(o[j]);
        // two operands: the order word is the key's byte offset
        if constexpr (K <= 2) {
#pragma unroll
            for (int j = 0; j < R; ++j) key[j] = *reinterpret_cast<const KeyT *>(kb + o[j]);
        }
    }

    // The counts of the workgroups before this one are asked for when the values are there: what decides is whether the words are
    // published by then, because one that is not costs a sleep and another round trip, and all workgroups poll the same few lines
    // (asked for together with the values, three vectors 63.8 us, three CSR matrices 89.5, two DCSR matrices of 20M 174; like this
    // 57.7, 83.3 and 159.6.  All of them looked up in parallel, seven wavefronts on the words of a chunk each, was slower still: 191).
    unsigned long long early_total = 0ull;
    auto ask_for_counts = [&]() {
        if (wave == 0) {
            const int m = (int)(p - chunk0);
#pragma unroll
            for (int i = 0; i < kWordLoads; ++i) {
                const int j = i * NACHO_WAVE + lane;
                early[i] = kWordValid;
                if (i * NACHO_WAVE < m && j < m)
                    early[i] = __hip_atomic_load(&counts_of[chunk0 + j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        } else if (wave == 1 && lane < chunk)
            early_total = __hip_atomic_load(&totals[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };

    // CSR: the rows whose pos this partition writes, and the places before such a row
    int first_row = 0, end_row = 0, pos_at = 0;
    auto places_before = [&](int row) {
        int m = 0;
#pragma unroll
        for (int t = 0; t < K; ++t) {
            if (t >= k) break;
            // (products of more operands: the pointer read again, not held from the staging on in scalar registers that move through
            // vector ones; five CSR matrices of 16M entries in all 104 to 101 us)
            const int at = (kMul && K > 2 ? pos_of(t, D - 1) : seg_pos[kWindow ? t : 0])[row] - of(q_v, t), len = of(len_v, t);
            m += at < 0 ? 0 : (at < len ? at : len);
        }
        return m;
    };
    if (FMT == SPADD_CSR) {
        first_row = row0 + (w.cont ? 1 : 0);
        end_row = table_coord(p + 1, 0) + (int)w.cont_next;
        if ((unsigned)first_row + (unsigned)tid < (unsigned)end_row) pos_at = places_before(first_row + tid);
    }

    // ---- the keys of the output entries, and what else the sums and products need ----------------
    // (past the last place: any words)
    auto load_keys = [&]() {
        if (__builtin_expect(far, 0)) {
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const int m = place0 + j * NACHO_WAVE + lane;
                key[j] = keys[w.order[m < n ? m : n - 1] & 0x1fff];
            }
        } else {
            const KeyT *first = keys + mb + place0 + lane;
#pragma unroll
            for (int j = 0; j < R; ++j) key[j] = first[j * NACHO_WAVE];
        }
    };
    // Products.  Few places are emitted, one in k at most and often one in ten, so the wavefront's emitted ones are moved together
    // first: the k places of an emitted entry hold the operands' entries in operand order, and behind each other the
    // order words of all such places are records of k words, one a lane.  What an output entry takes -- rows, addresses, values,
    // stores -- is then done once per 64 of them and not for every place (two DCSR matrices of 20M, one place in ten emitted: 135.8 to 112.8 us,
    // 130 to 85 vector instructions a place; two vectors of 8M with nearly all coordinates in both 62.3 to 52.0; two CSR matrices of 2.5M
    // 28.9 to 27.1).
    const int emitted = kMul ? of(wave_incl, NACHO_WAVE - 1) & 0xffff : 0;
    uint16_t *const records = w.order + (K <= 2 ? 0 : mb) + place0;
    int words_here = 0;                        // words of the records that lie in the wavefront's own places; the rest is in w.behind
    auto record = [&](int i, int g) -> int {   // the staged word of the g-th operand's entry of output entry i
        const int at = i * k + g;
        const unsigned o = *(at < words_here ? records + at : &w.behind[wave][at - words_here]);
        return K <= 2 ? (int)(o / KB) : (int)(o & 0x1fffu);
    };
    if constexpr (kMul) {
        if (emits) {
            const unsigned long long before = (unsigned long long)(unsigned)lane_before((int)(e >> 32), 0) << 32 |
                                              (unsigned)lane_before((int)(unsigned)e, 0);
            unsigned long long members = e;
#pragma unroll
            for (int g = 1; g < K; ++g)
                if (g < k) members |= e << g | before >> (64 - g);
            if (lane >= R) members = 0ull;
            const int count = __popcll(members), incl = dpp_scan_add(count);
            words_here = of(incl, NACHO_WAVE - 1);
            KeyT head_key[K > 2 ? R : 1];
            if (K > 2 && !far) {
#pragma unroll
                for (int j = 0; j < R; ++j) head_key[j] = keys[mb + place0 + j * NACHO_WAVE + lane];
            }
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const unsigned long long mj = lane_word(members, j);
                if (my_bit(mj)) records[of(incl - count, j) + lanes_below(mj)] = (uint16_t)product_words[j];
            }
            if (K > 2 && !far) {               // (more than two operands: the merge moved the keys, and these go where the entries go)
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    const unsigned long long ej = lane_word(e, j);
                    if (my_bit(ej)) keys[mb + place0 + (of(wave_incl - block_counts, j) & 0xffff) + lanes_below(ej)] = head_key[j];
                }
            }
            if (lane < K) w.behind[wave][lane] = (uint16_t)word_behind;
            wave_sync();
            // kBatch output entries a lane at a time
            auto multiply = [&](auto batch_tag) {
                constexpr int kBatch = decltype(batch_tag)::value, kGroup = K <= 4 ? K : 4;
                const unsigned last_row = kMapped ? (unsigned)row_extent() - 1u : 0u;      // (operands that are not sorted can name any)
                // (read from their lanes afresh: the scalar registers are not held from the start for this)
                int firsts_v = sb_v, starts_v = q_v, lengths_v = len_v;
                asm volatile("" : "+v"(firsts_v), "+v"(starts_v), "+v"(lengths_v));
                int entry[kBatch];
                unsigned row[kBatch];
#pragma unroll
                for (int i = 0; i < kBatch; ++i) {
                    const int x = i * NACHO_WAVE + lane;
                    entry[i] = x < emitted ? x : emitted - 1;
                    key[i] = K <= 2 || far ? keys[record(entry[i], 0)] : keys[mb + place0 + entry[i]];
                    row[i] = kMapped ? min((unsigned)row0 + (unsigned)row_field(key[i]), last_row) : 0u;
                }
#pragma unroll
                for (int g0 = 0; g0 < K; g0 += kGroup) {
                    int at[kGroup][kBatch];
                    T v[kGroup][kBatch];
#pragma unroll
                    for (int g = g0; g < g0 + kGroup; ++g)
                        if (g < k) {
                            const int first = of(firsts_v, g), final = first + of(lengths_v, g) - 1;
#pragma unroll
                            for (int i = 0; i < kBatch; ++i) {
                                // (of the operand for sure: repeated coordinates can put another's entry here)
                                at[g - g0][i] = max(first, min(record(entry[i], g), final)) + (of(starts_v, g) - first);
                                if constexpr (kMapped)
                                    at[g - g0][i] += ints(arg_ptr->ops.start[g])[row[i]] - pos_of(g, 1)[row[i]];
                            }
                        }
#pragma unroll
                    for (int g = g0; g < g0 + kGroup; ++g)
                        if (g < k) {
                            const NACHO_GLOBAL T *values = global_ptr<T>((unsigned long long)(uintptr_t)arg_ptr->vals.v[g]);
#pragma unroll
                            for (int i = 0; i < kBatch; ++i) v[g - g0][i] = values[at[g - g0][i]];
                        }
#pragma unroll
                    for (int g = g0; g < g0 + kGroup; ++g)
                        if (g < k) {
#pragma unroll
                            for (int i = 0; i < kBatch; ++i) val[i] = g == 0 ? v[g - g0][i] : val[i] * v[g - g0][i];
                        }
                }
            };
            if (emitted <= NACHO_WAVE) multiply(std::integral_constant<int, 1>());
            else multiply(std::integral_constant<int, NP>());
        }
    }
    if constexpr (!kMul) if (n > 0) {
        if constexpr (K > 2) load_keys();
        {
            // sums: the equal keys behind a head belong to the lanes after it, in operand order
            load_heads();
            unsigned long long x = e;          // the heads with g equal keys behind them
#pragma unroll 1
            for (int g = 1; g < k; ++g) {
                x &= shifted(eq, eq_next, g);
                const unsigned long long some = __ballot(x != 0ull && lane < R);
                if (some == 0ull) break;
                if (g == 1) {
                    // places behind the wavefront's last one
                    const int m = place0 + R * NACHO_WAVE + lane;
                    if (lane < k - 1 && m < n) tail = value_at(order_of(m));
                }
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    const unsigned long long xj = lane_word(x, j);
                    if (xj == 0ull) continue;  // (uniform)
                    asm volatile("");          // (a branch it stays: all of them without one need too many registers)
                    const T a = val[j], b = j + 1 < R ? val[j + 1 < R ? j + 1 : j] : tail;
                    T from;
                    if constexpr (K <= 2 && sizeof(T) == 4) from = next_lane(a, b);
                    else from = lane_at(lane < g ? b : a, (lane + g) & (NACHO_WAVE - 1));
                    val[j] = my_bit(xj) ? val[j] + from : val[j];       // (a head is nobody's equal key)
                }
            }
        }
    }

    ask_for_counts();

    // ---- 4. prefix sum, second half: wavefront 0 reads the counts of the workgroups before this one in its
    // chunk, wavefront 1 those of the chunks before
    if (wave == 0) {
        int b_nnz = 0, b_rows = 0, b_slices = 0, unused = 0;
        bool ok = sum_words<true, kWordLoads>(counts_of, chunk0, (int)(p - chunk0), early, lane, b_nnz, b_rows);
        if (kCsf && ok) ok = sum_words<false, kWordLoads>(counts_of2, chunk0, (int)(p - chunk0), early, lane, b_slices, unused);
        if (lane == 0) {
            if (ok && (p == chunk0 + kChunk - 1 || p == P - 1)) {
                __hip_atomic_store(&totals[chunk], kTotalValid | pack_counts(b_rows + own_rows, b_nnz + own_nnz),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (kCsf)
                    __hip_atomic_store(&totals2[chunk], kTotalValid | pack_counts(0, b_slices + own_slices),
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            w.base_nnz = b_nnz;
            w.base_rows = b_rows;
            w.base_slices = b_slices;
            if (!ok) w.gave_up = 1;
        }
    } else if (wave == 1) {
        int c_nnz = 0, c_rows = 0, c_slices = 0, unused = 0;
        bool ok = true;
        if (chunk > 0) {
            ok = sum_totals<kChunk>(totals, counts_of, chunk, lane, early_total, c_nnz, c_rows);
            if (kCsf && ok) ok = sum_totals<kChunk>(totals2, counts_of2, chunk, lane, 0ull, c_slices, unused);
        }
        if (lane == 0) {
            w.more_nnz = c_nnz;
            w.more_rows = c_rows;
            w.more_slices = c_slices;
            if (!ok) w.gave_up = 1;
        }
    }
    lds_barrier();
    const bool gave_up = __builtin_amdgcn_readfirstlane(w.gave_up) != 0;
    fresh();
    if (tid == 0) {
        const auto &out = arg_ptr->out;
        const int base_nnz = w.base_nnz + w.more_nnz, base_rows = w.base_rows + w.more_rows;
        const int base_slices = w.base_slices + w.more_slices;
        // a status once set to an error stays: the errors are ordered, the gravest wins
        if (gave_up) atomicMin(out.status, (int32_t)NACHO_ERR_HIP);
        else if (broken) atomicMin(out.status, (int32_t)NACHO_ERR_INVALID_ARG);
        if (p == P - 1 && !gave_up) {
            // totals, tails and the capacity verdict (the only writer of these words)
            const long long total_nnz = (long long)base_nnz + own_nnz;
            const long long total_rows = kRowHeads ? (long long)base_rows + own_rows
                                                   : (FMT == SPADD_CSR ? row_extent() : 1);
            const long long total_slices = (long long)base_slices + own_slices;
            bool fits = total_nnz <= out.cap_nnz && (FMT != SPADD_DCSR || total_rows <= out.cap_rows);
            if (kCsf) {
                // third-order tensors: {slices, fibres, entries}; the tails of the three pos arrays
                out.counts[0] = total_slices;
                out.counts[1] = total_rows;
                out.counts[2] = total_nnz;
                fits = fits && total_slices <= out.cap_rows && total_rows <= out.cap_fibres;
                out.pos0[0] = 0;
                out.pos0[1] = (int32_t)total_slices;
                if (total_slices <= out.cap_rows) out.pos1[total_slices] = (int32_t)total_rows;
                if (total_rows <= out.cap_fibres) out.pos2[total_rows] = (int32_t)total_nnz;
            } else {
                out.counts[0] = total_rows;
                out.counts[1] = total_nnz;
            }
            if (!fits) atomicMin(out.status, (int32_t)NACHO_ERR_CAPACITY);
            if (FMT == SPADD_VECTOR || kCoo) { out.pos1[0] = 0; out.pos1[1] = (int32_t)total_nnz; }
            if (FMT == SPADD_CSR) out.pos1[row_extent()] = (int32_t)total_nnz;
            if (FMT == SPADD_DCSR) {
                out.pos0[0] = 0;
                out.pos0[1] = (int32_t)total_rows;
                if (total_rows <= out.cap_rows) out.pos1[total_rows] = (int32_t)total_nnz;
            }
        }
    }
    const WaveLog wlog = {arg_ptr->wlog.rec, arg_ptr->wlog.capacity};
    auto log_end = [&]() { wave_end(wlog, (long long)p * kWaves + wave, stamp, logged_items, logged_rows); };
    if (gave_up) return log_end();             // no offset: nothing of this partition may be written

    // ---- 5. compute: write the partition's output ------------------------------
    // (the partition's offsets are uniform: the stores address base + a small per-lane offset)
    fresh();
    const auto &out = arg_ptr->out;
    const int at_nnz = __builtin_amdgcn_readfirstlane(w.base_nnz + w.more_nnz);
    const int at_rows = __builtin_amdgcn_readfirstlane(w.base_rows + w.more_rows);
    const int at_slices = __builtin_amdgcn_readfirstlane(w.base_slices + w.more_slices);
    auto room_of = [](int64_t cap, int at) {
        const int64_t left = cap - at;
        return left < 0 ? 0 : (left > 0x7fffffffll ? 0x7fffffff : (int)left);
    };
    const int room = room_of(out.cap_nnz, at_nnz);
    const int room_rows = kRowHeads ? room_of(kCsf ? out.cap_fibres : out.cap_rows, at_rows) : 0;
    const int room_slices = kCsf ? room_of(out.cap_rows, at_slices) : 0;
    const bool tight = own_nnz > room;         // (uniform: the capacity ends inside this partition or before it)
    if (FMT == SPADD_CSR) {
        // pos of every row that starts inside this partition: the output entries before its first place
        NACHO_GLOBAL int32_t *pos_out = global_out(out.pos1);
        const unsigned mine = (unsigned)first_row + (unsigned)tid;
        for (unsigned row = mine; row < (unsigned)end_row; row += kThreads) {
            const int m = row == mine ? pos_at : places_before((int)row);
            const int b = m / NACHO_WAVE;
            int before = own_nnz;
            if (b < NB) before = w.wave_before[b / R] + w.block_before[b] +
                                 __popcll(w.emitted[b] & low_bits(m & (NACHO_WAVE - 1)));
            pos_out[row] = at_nnz + before;
        }
    }
    // (32-bit byte offsets from a scalar base: a partition's output is far smaller than 4 GB)
    typedef NACHO_GLOBAL char *Out;
    auto out_at = [](auto *base, int first) -> Out { return (Out)(global_out(base) + first); };
    auto store = [](Out base, unsigned i, auto v) {
        *reinterpret_cast<NACHO_GLOBAL decltype(v) *>(base + i * (unsigned)sizeof(v)) = v;
    };
    const Out crd_out = out_at(kCsf ? out.crd2 : out.crd1, at_nnz), val_out = out_at(static_cast<T *>(out.val), at_nnz);
    const Out row_out = kCoo ? out_at(out.crd0, at_nnz) : nullptr;
    // rows (fibres): coordinate and start; slices: the same
    const Out seg_crd_out = kRowHeads ? out_at(kCsf ? out.crd1 : out.crd0, at_rows) : nullptr;
    const Out seg_pos_out = kRowHeads ? out_at(kCsf ? out.pos2 : out.pos1, at_rows) : nullptr;
    const Out top_crd = kCsf ? out_at(out.crd0, at_slices) : nullptr;
    const Out top_pos = kCsf ? out_at(out.pos1, at_slices) : nullptr;
    int at = wave_before & 0xffff, at_row = wave_before >> 16, at_slice = slices_before;
    const bool slices = kCsf && __ballot(lane < R && sl != 0ull) != 0ull;      // (few wavefronts' places start one)
    if constexpr (kMul) {
        if (kInstrument) {
            const int left = n - place0;
            logged_items += left >= R * NACHO_WAVE ? R * NACHO_WAVE : (left > 0 ? left : 0);
        }
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            if (j * NACHO_WAVE >= emitted) break;      // (uniform)
            const int x = j * NACHO_WAVE + lane, loc = at + x;
            if (x < emitted && (!tight || loc < room)) {
                store(crd_out, (unsigned)loc, (int32_t)(D == 1 ? (uint32_t)key[j] : (uint32_t)(key[j] & col_mask)));
                if (kCoo) store(row_out, (unsigned)loc, row0 + (int32_t)(uint32_t)row_field(key[j]));
                store(val_out, (unsigned)loc, val[j]);
            }
        }
        if constexpr (D >= 2)
            if (__builtin_expect(far, 0)) {
                // (uniform, rare) the columns, whose lower bits the keys lack
#pragma unroll 1
                for (int x = lane; x < emitted; x += NACHO_WAVE) {
                    const int s = record(x, 0), col = column_at(0, s, row_field(keys[s]));
                    if (at + x < room) store(crd_out, (unsigned)(at + x), (int32_t)col);
                }
            }
    } else
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const unsigned long long ej = lane_word(e, j);
        if (kInstrument) {
            const int left = n - place0 - j * NACHO_WAVE;
            logged_items += left >= NACHO_WAVE ? NACHO_WAVE : (left > 0 ? left : 0);
            if (kRowHeads) logged_rows += (uint32_t)__popcll(lane_word(r, j));
        }
        const unsigned loc = (unsigned)(at + lanes_below(ej));
        unsigned long long stored = ej;
        if (__builtin_expect(tight, 0)) stored &= __ballot((int)loc < room);
        if (my_bit(stored)) {
            store(crd_out, loc, (int32_t)(D == 1 ? (uint32_t)key[j] : (uint32_t)(key[j] & col_mask)));
            if (kCoo) store(row_out, loc, row0 + (int32_t)(uint32_t)row_field(key[j]));
            store(val_out, loc, val[j]);
        }
        if constexpr (kRowHeads) {
            const unsigned long long rj = lane_word(r, j);
            if (rj != 0ull) {                  // (uniform)
                const unsigned rloc = (unsigned)(at_row + lanes_below(rj));
                const KeyT field = row_field(key[j]);
                if (my_bit(rj) && (int)rloc < room_rows) {
                    // (a row's coordinate; a fibre's j) and where its entries start
                    store(seg_crd_out, rloc, kCsf ? (int32_t)(uint32_t)(field & ((KeyT(1) << jb) - KeyT(1))) : row0 + (int32_t)(uint32_t)field);
                    store(seg_pos_out, rloc, at_nnz + (int)loc);
                }
                if (kCsf && slices) {
                    const unsigned long long sj = lane_word(sl, j);
                    const unsigned sloc = (unsigned)(at_slice + lanes_below(sj));
                    if (my_bit(sj) && (int)sloc < room_slices) {
                        store(top_crd, sloc, row0 + (int32_t)(uint32_t)(field >> jb));
                        store(top_pos, sloc, at_rows + (int)rloc);
                    }
                    at_slice += __popcll(sj);
                }
                at_row += __popcll(rj);
            }
        }
        at += __popcll(ej);
    }
    if constexpr (D >= 2 && !kMul)
        if (__builtin_expect(far, 0)) {
            // (uniform, rare) the columns, whose lower bits the keys lack
            at = wave_before & 0xffff;
#pragma unroll 1
            for (int j0 = 0; j0 < R && place0 + j0 * NACHO_WAVE < n; j0 += 4) {
                int col[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int m = place0 + (j0 + i) * NACHO_WAVE + lane;
                    int t;
                    const int s = word_of(w.order[m < n ? m : n - 1], t);
                    col[i] = column_at(t, s, row_field(keys[s]));
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const unsigned long long ej = j0 + i < R ? lane_word(e, j0 + i) : 0ull;
                    const int loc = at + lanes_below(ej);
                    if (my_bit(ej) && loc < room) store(crd_out, (unsigned)loc, (int32_t)col[i]);
                    at += __popcll(ej);
                }
            }
        }
    log_end();
}

// Four workgroups run on a compute unit if a wavefront takes no more than 64 vector and 80 scalar registers.  The search of a workgroup's
// own boundaries asks for more of both (67 to 73, 82 to 106): three run, and calls of 769 to 1024 partitions take a second round (four vectors
// of 4.2M fp32 entries in all: 47.5 us, held to the registers of four 37.4).  Held to them, long partitions of doubles spill from four operands
// on, and five and more operands move scalars through vector registers (0.3M to 3.3M entries 4 to 7 % slower): these have a
// kernel for middle partitions beside the one for three workgroups, for calls that three a compute unit do not hold (five vectors of 4.2M 62.4
// to 48.5 us).
template <typename T, int K> constexpr bool kSearchOfFour = K <= (sizeof(T) == 8 ? 3 : 4);

template <int FMT, typename T, typename KeyT, int kSize, int K, bool kMul, bool kMapped, bool kSearch = false>
__global__ void __launch_bounds__(kThreads, (kSearch && kSize == MERGE_LONG && !kSearchOfFour<T, K> ? 2 : 8))
spadd_kernel(MergeArgs args)
{
    __shared__ TileOf<FMT, T, KeyT, kSize> w;
    const WaveStamp stamp = wave_begin();
    // (not where half of the workgroups find that they have nothing to do)
    if constexpr (!kMapped) touch_arguments<sizeof(MergeArgs) <= 1408 ? sizeof(MergeArgs) : 1408>();
    const ArgPtr arg_ptr = (ArgPtr)__builtin_amdgcn_kernarg_segment_ptr();
    merge_partition<FMT, T, KeyT, kSize, K, kMul, kMapped, kSearch>(arg_ptr, w, args.ops, stamp);
}

inline int64_t chunks_of(int64_t P, int chunk) { return (P + chunk - 1) / chunk; }

template <int FMT, typename T, typename KeyT, int kSize, int K, bool kMul, bool kMapped, bool kSearch>
hipError_t launch_k(const MergeLaunch &a)
{
    MergeArgs args{a.ops, a.vals, a.P, chunks_of(a.P, chunk_size(FMT, kMul)), a.coord, a.posn, a.tile_state, a.out, a.fields,
                   nacho_host::wave_log(), a.search};
    constexpr int kRun = kSearch && sizeof(T) == 4 && kSearchOfFour<T, K> ? (int)MERGE_LONG : kSize;    // (floats: that one does as well)
    hipLaunchKernelGGL((spadd_kernel<FMT, T, KeyT, kRun, K, kMul, kMapped, kSearch>), dim3((unsigned)a.P), dim3(kThreads), 0,
                       a.s, args);
    return hipGetLastError();
}

// instantiated for up to 2, 3, 4 and 8 operands: the per-entry loops over the runs are unrolled
template <int FMT, typename T, typename KeyT, int kSize, bool kMul, bool kMapped, bool kSearch>
hipError_t launch_one(const MergeLaunch &a)
{
    if (a.ops.k <= 2) return launch_k<FMT, T, KeyT, kSize, 2, kMul, kMapped, kSearch>(a);
    if (a.ops.k <= 3) return launch_k<FMT, T, KeyT, kSize, 3, kMul, kMapped, kSearch>(a);
    if (a.ops.k <= 4) return launch_k<FMT, T, KeyT, kSize, 4, kMul, kMapped, kSearch>(a);
    return launch_k<FMT, T, KeyT, kSize, 8, kMul, kMapped, kSearch>(a);
}

template <int FMT, bool kMul, bool kMapped = false, bool kSearch = false>
hipError_t launch_types(int dtype, const MergeLaunch &a)
{
    if constexpr (FMT != SPADD_VECTOR)
        if (a.fields.wide) {
            if (dtype == NACHO_F64) return launch_one<FMT, double, uint64_t, MERGE_LONG, kMul, kMapped, kSearch>(a);
            return launch_one<FMT, float, uint64_t, MERGE_LONG, kMul, kMapped, kSearch>(a);
        }
    if constexpr (!kSearch)
        if (a.fields.size == MERGE_SHORT) {
            if (dtype == NACHO_F64) return launch_one<FMT, double, uint32_t, MERGE_SHORT, kMul, kMapped, kSearch>(a);
            return launch_one<FMT, float, uint32_t, MERGE_SHORT, kMul, kMapped, kSearch>(a);
        }
    if (kMapped || a.fields.size == MERGE_MIDDLE) {
        if (dtype == NACHO_F64) return launch_one<FMT, double, uint32_t, MERGE_MIDDLE, kMul, kMapped, kSearch>(a);
        return launch_one<FMT, float, uint32_t, MERGE_MIDDLE, kMul, kMapped, kSearch>(a);
    }
    if constexpr (!kMapped) {
        if (dtype == NACHO_F64) return launch_one<FMT, double, uint32_t, MERGE_LONG, kMul, kMapped, kSearch>(a);
        return launch_one<FMT, float, uint32_t, MERGE_LONG, kMul, kMapped, kSearch>(a);
    }
    return hipErrorInvalidValue;               // (not reached)
}

}  // namespace

}  // namespace nacho
