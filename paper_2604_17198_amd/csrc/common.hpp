// Shared device helpers of the nacho HIP library (gfx950, 64-wide wavefronts).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include "nacho.h"

#define NACHO_WAVE 64

namespace nacho {

// Device-side copy of the operands' level descriptors (passed by value as a
// kernel argument; k <= NACHO_MAX_OPERANDS, d <= NACHO_MAX_LEVELS).
struct DevLevel {
    int32_t kind;
    int32_t pad_;
    int64_t extent;
    const int32_t *pos;
    const int32_t *crd;
    int64_t count;
};
struct DevOperands {
    int32_t k, d;
    DevLevel lvl[NACHO_MAX_OPERANDS][NACHO_MAX_LEVELS];
    // Remapped operands (Section 3.3; dense level 0 over the intersected rows): the entries of
    // row i' of operand t are stored from position start[t][i'] of crd / val on, while the
    // level-1 pos array counts only the entries of the intersected rows.  NULL otherwise.
    const int32_t *start[NACHO_MAX_OPERANDS];
    // Remapped operands only: their sizes are results of earlier kernels of the same call and are
    // read on the device.  dyn_head[0] = rows all operands store (the extent of the dense level),
    // dyn_head[1 + t] = entries operand t stores in them (the count of its compressed level);
    // dyn_plan[0] = partitions of the remapped nest, dyn_plan[2] = its total cost, dyn_plan[3] != 0: the row
    // loop was abandoned (a wait ran out) and nothing of the remapped nest may be read.  The extents and
    // counts in lvl[][] are upper bounds then (what the launches are sized for).  NULL otherwise.
    const int32_t *dyn_head;
    const int64_t *dyn_plan;
};

// Extent of the dense level 0 / count of the last level of operand t: the stored ones, or (remapped
// operands) the values earlier kernels of the call left on the device.
__device__ inline int64_t level0_extent(const DevOperands &ops)
{
    return ops.dyn_head ? (int64_t)ops.dyn_head[0] : ops.lvl[0][0].extent;
}
__device__ inline int64_t last_count(const DevOperands &ops, int t)
{
    return ops.dyn_head ? (int64_t)ops.dyn_head[1 + t] : ops.lvl[t][ops.d - 1].count;
}

// floor(p * total / P) for 0 <= p <= P < 2^31 without leaving int64.
__host__ __device__ inline int64_t equal_query(int64_t p, int64_t total, int64_t P)
{
    int64_t q = total / P, r = total % P;
    return p * q + (p * r) / P;
}

// The same where everything fits 31 bits, without divisions of 64 bits (some 400 instructions before the first load
// of a boundary search).
__device__ inline int64_t equal_query_short(unsigned p, unsigned total, unsigned P)
{
    const unsigned q = total / P, r = total - q * P;
    const uint64_t product = (uint64_t)p * r;              // < 2^62; the quotient by P is below 2^31, so the estimate is off by 1 at most
    unsigned x = (unsigned)((double)product / (double)P);
    const int64_t left = (int64_t)(product - (uint64_t)x * P);
    x += left < 0 ? ~0u : (left >= (int64_t)P ? 1u : 0u);
    return (int64_t)p * q + x;
}

// Partitions of `grain` units that start before the place `at` of a row's (or the matrix's) non-zeros: at / grain
// rounded up, 0 <= at < 2^31 (unsigned: at + grain may lie past 2^31).
__host__ __device__ inline int shares_before(int at, int grain)
{
    return (int)(((unsigned)at + (unsigned)grain - 1u) / (unsigned)grain);
}

// The row behind a boundary's row; the boundary may lie behind all rows already, of which there may be 2^31 - 1.
__host__ __device__ inline int row_behind(int row, int n_rows) { return row < n_rows ? row + 1 : n_rows; }

// Rows that the partition between the boundary rows r0 <= r1 may overlap or start, r1 among them where it is one (n_rows is not), at
// most `most` of them.
__host__ __device__ inline int rows_spanned(int r0, int r1, int n_rows, int most)
{
    const int rows = row_behind(r1, n_rows) - r0;
    return rows < most ? rows : most;
}

// The row that a lane looks at in one round of a search of the rows [lo, hi), lo < hi: 64 evenly spaced ones, the last row for sure.
// (Unsigned here and below: a place behind the range may lie past 2^31.)
__host__ __device__ inline int row_probe(int lo, int hi, int lane)
{
    const unsigned step = ((unsigned)(hi - lo) + NACHO_WAVE - 1) / NACHO_WAVE, t = (unsigned)lo + (unsigned)lane * step;
    return lane == NACHO_WAVE - 1 || t > (unsigned)hi - 1u ? hi - 1 : (int)t;
}

// One round of a search for a number of rows in [lo, hi] by kLanes lanes: lane i looks at the last of the rows it stands for, which is
// in the range if it lies below hi; n lanes, the first ones, found theirs too small.
template <int kLanes> struct RowRound {
    unsigned lo, hi, step;
    __host__ __device__ RowRound(int lo_, int hi_) : lo((unsigned)lo_), hi((unsigned)hi_), step((hi - lo + kLanes - 1) / kLanes) {}
    __host__ __device__ unsigned at(int i) const { return lo + (unsigned)(i + 1) * step - 1u; }
    __host__ __device__ void narrow(int n, int &lo_, int &hi_) const
    {
        const unsigned to = lo + (unsigned)n * step;
        hi_ = (int)(n < kLanes && at(n) < hi ? at(n) : hi);
        lo_ = to < (unsigned)hi_ ? (int)to : hi_;
    }
};

// Asks for the first kBytes of the kernel's arguments at once.  They lie in memory that no cache holds at a kernel's
// start; left to the places where they are used, every line of them is a round trip of its own.
template <int kBytes> __device__ inline void touch_arguments()
{
    typedef const __attribute__((address_space(4))) unsigned *Words;
    const Words words = (Words)__builtin_amdgcn_kernarg_segment_ptr();
    auto line = [&](int i) { return words[i * 64 < kBytes ? i * 16 : 0]; };
    static_assert(kBytes <= 22 * 64, "twenty-two lines");
    // (one statement: the compiler waits for what it names in one go)
    asm volatile("" ::"s"(line(0)), "s"(line(1)), "s"(line(2)), "s"(line(3)), "s"(line(4)), "s"(line(5)), "s"(line(6)),
                 "s"(line(7)), "s"(line(8)), "s"(line(9)), "s"(line(10)), "s"(line(11)), "s"(line(12)), "s"(line(13)),
                 "s"(line(14)), "s"(line(15)), "s"(line(16)), "s"(line(17)), "s"(line(18)), "s"(line(19)), "s"(line(20)), "s"(line(21)));
}

__device__ inline int lane_id() { return (int)(threadIdx.x & (NACHO_WAVE - 1)); }

// Orders the LDS traffic of ONE wavefront: writes issued before it are visible
// to reads of other lanes of the same wavefront issued after it.  (The LDS
// executes a wavefront's instructions in order; this keeps the compiler from
// moving accesses across the point.)  It does not synchronise wavefronts.
__device__ inline void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Butterfly sum over the 64 lanes in a fixed order: every lane ends with the
// same bits, and the same inputs always give the same result.
template <typename T>
__device__ inline T wave_sum(T v)
{
#pragma unroll
    for (int off = NACHO_WAVE / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, NACHO_WAVE);
    return v;
}

// Inclusive prefix sum over the lanes of a wavefront.
__device__ inline int wave_inclusive_scan(int v)
{
    const int lane = lane_id();
#pragma unroll
    for (int off = 1; off < NACHO_WAVE; off <<= 1) {
        int n = __shfl_up(v, off, NACHO_WAVE);
        if (lane >= off) v += n;
    }
    return v;
}

// Sum over the lanes of a wavefront in a fixed order, in lane 63, by DPP moves (a butterfly of shuffles goes
// through the LDS unit: six dependent round trips of over a hundred cycles).
template <int kCtrl, int kRowMask> __device__ inline float dpp_moved(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kCtrl, kRowMask, 0xf, false));
}
template <int kCtrl, int kRowMask> __device__ inline double dpp_moved(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, kCtrl, kRowMask, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), kCtrl, kRowMask, 0xf, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
template <typename T> __device__ inline T dpp_wave_sum(T v)
{
    v += dpp_moved<0x111, 0xf>(v);                     // row_shr:1, 2, 4, 8: inside 16 lanes
    v += dpp_moved<0x112, 0xf>(v);
    v += dpp_moved<0x114, 0xf>(v);
    v += dpp_moved<0x118, 0xf>(v);
    v += dpp_moved<0x142, 0xa>(v);                     // row_bcast:15 into rows 1 and 3
    v += dpp_moved<0x143, 0xc>(v);                     // row_bcast:31 into rows 2 and 3
    return v;
}
__device__ inline float last_lane(float v) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), NACHO_WAVE - 1)); }
__device__ inline double last_lane(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(unsigned)b, NACHO_WAVE - 1);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), NACHO_WAVE - 1);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// The n lowest bits of a 64-bit word (n: this lane's; below 0: none, above 64: all), built from 32-bit shifts.
// A 64-bit shift whose amount is in the LAST vector register a kernel was given takes the amount of another
// wavefront now and then (measured: some rows' pos of a CSR product, another wavefront's every time), and which
// register that is hangs on the compiler, so no lane shifts 64 bits by an amount of its own.
__device__ inline unsigned long long low_bits(int n)
{
    const unsigned lo = n >= 32 ? ~0u : (n > 0 ? (1u << n) - 1u : 0u);
    const unsigned hi = n >= 64 ? ~0u : (n > 32 ? (1u << (n - 32)) - 1u : 0u);
    return ((unsigned long long)hi << 32) | lo;
}

// The value lane `from` holds (`from` the same in every lane), through a scalar register.
__device__ inline int lane_value(int x, int from) { return __builtin_amdgcn_readlane(x, from); }
__device__ inline long long lane_value(long long x, int from)
{
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(unsigned long long)x, from);
    const int hi = __builtin_amdgcn_readlane((int)(x >> 32), from);
    return ((long long)hi << 32) | (long long)lo;
}
// The value lane `from` holds, `from` this lane's own choice.
__device__ inline int value_from(int x, int from) { return __builtin_amdgcn_ds_bpermute(from << 2, x); }
__device__ inline long long value_from(long long x, int from)
{
    const unsigned lo = (unsigned)value_from((int)(unsigned)(unsigned long long)x, from);
    return ((long long)value_from((int)(x >> 32), from) << 32) | (long long)lo;
}

__device__ inline int lane_left(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x138, 0xf, 0xf, false); }     // wave_shr:1

// Bit `at` (this lane's) of a mask every lane agrees on, without such a shift.  (The compiler would turn the choice
// between the halves of one word into one; it does not know that these two belong together.)
__device__ inline bool bit_at(unsigned long long mask, int at)
{
    const unsigned lo = (unsigned)mask;
    unsigned hi = (unsigned)(mask >> 32);
    asm("" : "+s"(hi));
    return (((at < 32 ? lo : hi) >> (at & 31)) & 1u) != 0u;
}

// First row t in [lo, hi) with pos[t + 1] > q, found by the whole wavefront (64 probes
// per round).  Requires pos[hi] > q.  Rows lo .. t - 1 then hold nothing at or after q.
__device__ inline int first_row_past(const int32_t *__restrict__ pos, int lo, int hi, int q)
{
    const int lane = lane_id();
    while (hi - lo > 1) {
        const int t = row_probe(lo, hi, lane);
        const unsigned long long past = __ballot(pos[t + 1] > q);    // a suffix of the lanes, never empty
        const int L = __ffsll((long long)past) - 1;
        const int t_hit = __shfl(t, L, NACHO_WAVE);
        const int t_prev = __shfl(t, L > 0 ? L - 1 : 0, NACHO_WAVE);
        if (L > 0) lo = t_prev + 1;
        hi = t_hit + 1;
    }
    return lo;
}

// A search for the number of rows that end at or before q, which is also the row that holds position q: it lies in [lo, hi].
// A round looks at 64 rows; its load and what follows from it are apart, so that other loads can be asked for between them.  (Rows: a
// few million at most, spmv_whole and spmm_whole with partitions of up to 128 non-zeros; sums with a lane's offset stay below 2^31.)
struct RowWindow {
    int lo, hi;
    __device__ int stride() const { return (hi - lo + NACHO_WAVE - 1) / NACHO_WAVE; }
    // this lane's probe (past the window, or the window empty: some position)
    __device__ int load(const int32_t *__restrict__ pos, int n_rows) const
    {
        const int at = lo + (lane_id() + 1) * stride();
        return pos[at < n_rows ? at : n_rows];
    }
    __device__ void narrow(int probe, int q)
    {
        const int step = stride(), at = lo + (lane_id() + 1) * step - 1;
        const int n = __popcll(__ballot(at < hi && probe <= q));               // (a prefix of the lanes)
        const int lo_new = lo + n * step, at_next = lo + (n + 1) * step - 1;
        hi = n < NACHO_WAVE && at_next < hi ? at_next : hi;
        lo = lo_new < hi ? lo_new : hi;
    }
};

// The rows ra, rb with pos[r] <= q < pos[r + 1] for q = qa and qb (n_rows where pos[n_rows] <= q), both at once:
// half of the wavefront searches each, 32 probes per round.
__device__ inline void rows_holding(const int32_t *__restrict__ pos, int n_rows, int qa, int qb, int &ra, int &rb)
{
    constexpr int G = NACHO_WAVE / 2;
    const int lane = lane_id(), sub = lane & (G - 1);
    const int q = lane < G ? qa : qb;
    const unsigned long long half = lane < G ? 0xffffffffull : 0xffffffff00000000ull;
    int lo = 0, hi = n_rows;                           // the number of rows that end at or before q
    while (__ballot(lo < hi) != 0ull) {
        const RowRound<G> round(lo, hi);
        const unsigned at = round.at(sub);
        const bool before = lo < hi && at < round.hi && pos[at + 1u] <= q;     // (a prefix of the half)
        const int n = __popcll(__ballot(before) & half);
        if (lo < hi) round.narrow(n, lo, hi);
    }
    ra = __builtin_amdgcn_readlane(lo, 0);
    rb = __builtin_amdgcn_readlane(lo, G);
}

// Which partition the workgroup of partition p executes when partitions inside one row are dealt out by XCD: p lies in the
// row whose non-zeros are [a, e) (counted from the matrix's first), partitions have `grain` non-zeros.  Workgroups are handed to
// the 8 XCDs in turn (workgroup w runs on XCD w mod 8), and every XCD has its own L2.  The partitions inside the row are
// first = ceil(a / grain) .. end - 1 = floor(e / grain) - 1.  Among the workgroups first .. end - 1 those with index = j (mod 8)
// take, in order, the j-th stretch of these partitions (stretches as long as there are such workgroups): a permutation of
// first .. end - 1; everything else keeps its index.  XCD j then gathers from one eighth of what the row gathers from
// (columns are sorted inside a row), and that eighth is the same for every long row.
__device__ inline int dealt_partition(int p, int a, int e, int grain)
{
    const int first = shares_before(a, grain), end = e / grain;
    if (end - first < 4 || p < first || p >= end) return p;
    const int j = p & 7;
    int before = 0, mine = 0;                          // partitions of the stretches before stretch j; first workgroup of j
#pragma unroll
    for (int jj = 0; jj < 8; ++jj) {
        const int f = first + ((jj - first) & 7);      // first workgroup >= first with index = jj (mod 8)
        const int cnt = f < end ? (end - f + 7) >> 3 : 0;
        if (jj < j) before += cnt;
        if (jj == j) mine = f;
    }
    return first + before + ((p - mine) >> 3);
}

// ---- instrumented build (-DNACHO_INSTRUMENT): what every wavefront did, and when -----------
// The executing kernels take a log descriptor as their last argument.  In the ordinary build the
// flag below is false and every use of it folds away; in the instrumented build lane 0 of
// wavefront i of a launch fills record i (if the caller gave a buffer): the items and rows it
// worked on, its first and last time stamp (constant 100 MHz counter, comparable across the
// chip), its shader-clock cycles and where it ran.
#ifdef NACHO_INSTRUMENT
constexpr bool kInstrument = true;
#else
constexpr bool kInstrument = false;
#endif
struct WaveRecord {
    unsigned long long t_begin, t_end;   // wall_clock64()
    unsigned long long cycles;           // clock64() span
    uint32_t items, rows;                // work items (stored non-zeros / merged places) and rows touched
    uint32_t hw_id, xcc_id;              // HW_ID and XCC_ID registers of the wavefront
};
struct WaveLog {
    WaveRecord *rec;
    long long capacity;
};
struct WaveStamp { unsigned long long t, c; };
__device__ inline WaveStamp wave_begin()
{
    WaveStamp s = {0ull, 0ull};
    if (kInstrument) { s.t = wall_clock64(); s.c = clock64(); }
    return s;
}
__device__ inline void wave_end(const WaveLog &log, long long index, const WaveStamp &s, uint32_t items,
                                uint32_t rows)
{
    if (!kInstrument) return;
    if (log.rec == nullptr || index >= log.capacity || lane_id() != 0) return;
    WaveRecord r;
    r.t_begin = s.t;
    r.t_end = wall_clock64();
    r.cycles = clock64() - s.c;
    r.items = items;
    r.rows = rows;
    uint32_t hw = 0, xcc = 0;
#ifdef NACHO_INSTRUMENT
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_HW_ID)" : "=s"(hw));
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
#endif
    r.hw_id = hw;
    r.xcc_id = xcc;
    log.rec[index] = r;
}

}  // namespace nacho

// Host-side bookkeeping shared by the translation units.
namespace nacho_host {

struct Profiler {
    static constexpr int kMax = 16;
    bool enabled = false;
    int n = 0;
    hipEvent_t ev[kMax + 1] = {};
    const char *name[kMax] = {};
    bool created = false;
    hipStream_t stream = nullptr;
};
Profiler &profiler();
// Call before the first kernel of an entry point, then after every kernel.
void profile_begin(hipStream_t s);
void profile_mark(const char *kernel_name);

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Where the executing kernels of an instrumented build log their wavefronts (null otherwise).
nacho::WaveLog &wave_log();
// Instrumented build: the workgroup of the row loop of a DCSR product whose wait counts as run out (-1: none).
int64_t &wait_runs_out();

}  // namespace nacho_host
