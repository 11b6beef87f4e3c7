// Recursive partitioning (Section 3.3, Algorithm 2) for a product whose OUTER
// level is a sparse intersection: the Hadamard product of k DCSR matrices.
//
// Hierarchical skipping (rows that not every operand stores are never
// coiterated) makes the plain non-zero count of Section 4.2.2 the wrong cost,
// so the row loop is run first, on its own partitions, and memoises the cost
// of the loop below it:
//   1. the rows all operands store are found (a k-way intersection of the
//      level-0 coordinate arrays, partitioned by Algorithm 1 on those arrays);
//   2. for the i'-th such row, T[i'] = C_j(N_j | i) is stored -- here per
//      operand, S_t[i'] = number of entries operand t stores in the row, so that
//      T = sum_t S_t -- together with the position of the row's first entry in
//      every operand;
//   3. exclusive prefix sums turn S_t into the remapped cost function
//      C'_i(x) = T'[x] = sum_t S_t'[x].
// The remapped nest (i' dense over the intersected rows, then the column
// intersection) has no skipping left: it is what the partition kernel and the
// merge kernel run on, each operand seen as a CSR matrix over i' whose pos
// array is S_t' and whose row i' starts at the stored position in crd/val.
// Finally the rows of the result that received no entry are dropped.
//
// What bounds it: the arrays are short (a few hundred thousand rows), so the stage is a chain of latencies and kernel
// launches.  All of 1. to 3. is one kernel, one workgroup per partition of the level-0 arrays: their segments are
// staged in LDS and searched there, and the prefix sums (number of rows, S_t per operand) run along the workgroups by
// decoupled look-back.  As kernels of their own -- match, two scans of two kernels each, plan -- with 4096 items per
// workgroup these took 56 of the 226 us of a product of two matrices of 20M entries in 100k rows.  The rows without
// an entry are dropped by a scan of the same kind (one kernel instead of two, 18 us).
#include "common.hpp"
#include "kernels.hpp"

namespace nacho {

namespace {

constexpr int kScanThreads = 256, kScanWaves = kScanThreads / NACHO_WAVE;

// ---- prefix sums along the workgroups of a launch (decoupled look-back) --------
// Workgroup p publishes its own sum (an aggregate), reads back over the words of the workgroups before it until it
// meets one that already knows the sum of everything up to and including itself (a prefix), and publishes its own
// prefix.  Workgroups are handed out in index order and wait only for smaller indexes, so the waits end (they are
// bounded all the same).
constexpr unsigned long long kAggregate = 1ull << 62, kPrefix = 1ull << 63;
constexpr int kSpinLimit = 1 << 14;

__device__ inline void publish(unsigned long long *state, int64_t p, unsigned long long flag, int v)
{
    __hip_atomic_store(&state[p], flag | (unsigned)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// By a whole wavefront: the sum of the workgroups before p, whose own sum is `own`; publishes the prefix.  A lane holds
// kWords words, all in flight at once: with a few hundred workgroups, which all start together and so find no prefix near, one
// trip to memory in place of one for every 64 of them.
constexpr int kWords = 4;
__device__ inline bool look_back(unsigned long long *state, int64_t p, int own, int &before)
{
    const int lane = lane_id();
    int sum = 0;
    bool done = p == 0;
    for (int64_t end = p; !done; end -= kWords * NACHO_WAVE) {         // words end - 1 - (64 u + lane)
        unsigned long long s[kWords], prefixes[kWords];
        for (int spins = 0;; ++spins) {
#pragma unroll
            for (int u = 0; u < kWords; ++u) {
                const int64_t j = end - 1 - (u * NACHO_WAVE + lane);
                s[u] = __hip_atomic_load(&state[j < 0 ? 0 : j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            bool waits = false, behind = false;        // (behind a prefix nothing counts)
#pragma unroll
            for (int u = 0; u < kWords; ++u) {
                if (end - 1 - (u * NACHO_WAVE + lane) < 0) s[u] = kPrefix;
                prefixes[u] = __ballot((s[u] & kPrefix) != 0ull);
                const unsigned long long missing = __ballot(s[u] == 0ull);
                // (lanes nearer than the nearest prefix count)
                const unsigned long long nearer = prefixes[u] ? (prefixes[u] & (0ull - prefixes[u])) - 1ull : ~0ull;
                waits = waits || (!behind && (missing & nearer) != 0ull);
                behind = behind || prefixes[u] != 0ull;
            }
            if (!waits) break;
            if (spins > kSpinLimit) return false;
            __builtin_amdgcn_s_sleep(4);
        }
#pragma unroll
        for (int u = 0; u < kWords; ++u) {
            const int nearest = prefixes[u] ? __ffsll((long long)prefixes[u]) - 1 : NACHO_WAVE - 1;
            const int part = wave_inclusive_scan(lane <= nearest ? (int)(unsigned)s[u] : 0);
            sum += done ? 0 : __builtin_amdgcn_readlane(part, NACHO_WAVE - 1);
            done = done || prefixes[u] != 0ull;
        }
    }
    before = sum;
    if (lane == 0) publish(state, p, kPrefix, sum + own);
    return true;
}

// ---- the row loop -----------------------------------------------------------
struct RowArrays {
    int32_t k;
    const int32_t *crd0[NACHO_MAX_OPERANDS], *pos1[NACHO_MAX_OPERANDS];
    int64_t runs_out;                                  // (instrumented build) the workgroup whose wait counts as run out
};

// What the kernels after the row loop need to know, left where they can read it: the number of
// partitions of the remapped nest (the rule of the fused calls: enough partitions that one fits a
// workgroup, a whole number of rounds of resident workgroups where that is near, at least what the caller asked for),
// the number of intersected rows and the remapped total cost.
struct PlanRule {
    int64_t capacity, round, P_min, P_max;
    __device__ void write(int64_t rows, int64_t total, int64_t *plan) const
    {
        int64_t need = total > 0 ? (total + capacity - 1) / capacity : 1;
        if (P_min == 0) need = whole_rounds(need, round);
        int64_t P = P_min > need ? P_min : need;
        if (P > P_max) P = P_max;
        plan[0] = P;
        plan[1] = rows;
        plan[2] = total;
    }
};

// One workgroup per partition of the level-0 coordinate arrays (at most kRemapGrain + k - 1 coordinates).  Equal
// coordinates of different operands fall in one partition (Section 6), so every row of operand 0 in the partition
// looks for itself in the partition's segment of every other operand.
//
// A chain of latencies: two trips to memory (the segments' places, then the rows and where their entries start together, all
// loads of a thread at once), searches in LDS side by side, the look-back.  (Operand by operand and row by row, with the starts
// asked for once the intersected rows are known and a trip for every 64 workgroups that the sums go back over: two matrices of 100k
// rows 13.3 us, so 10.7; the whole product of 15k entries each 29.7 us, so 27.8, of 20M each 105.5, so 102.4.)  K: the most
// operands.
template <int K>
__global__ void __launch_bounds__(kScanThreads)
remap_rows_kernel(RowArrays in, const int32_t *__restrict__ posn0, int64_t P0, RemapArrays r,
                  unsigned long long *__restrict__ state, PlanRule rule, int64_t *__restrict__ plan,
                  int32_t *__restrict__ status)
{
    constexpr int kFewest = K == 2 ? 2 : K - 1;                // operands of a call
    constexpr int kMost = kRemapGrain + K, kPairs = (kRemapGrain + kFewest - 1) / kFewest;     // coordinates, intersected rows of a partition
    constexpr int kEach = (kPairs + kScanThreads - 1) / kScanThreads, kLoads = (kMost + K + kScanThreads - 1) / kScanThreads;
    static_assert(kMost < (1 << 16), "places in a partition fit 16 bits");
    __shared__ int s_crd[kMost], s_pos[kMost + K];             // the rows of all operands; where their entries start (and the last one's end)
    __shared__ uint16_t s_q[K][kMost];                         // place of operand 0's row in the other operands' segments
    __shared__ uint16_t s_item[kPairs];                        // the intersected rows of the partition
    __shared__ int s_count[kScanWaves], s_len[K][kScanWaves], s_base[K + 1];
    __shared__ int s_fail;
    touch_arguments<sizeof(RowArrays) + sizeof(RemapArrays) + sizeof(PlanRule) + 40>();
    const int tid = threadIdx.x, lane = lane_id(), wave = tid / NACHO_WAVE, k = K == 2 ? 2 : in.k;
    const int64_t p = blockIdx.x;

    int lo[K], off[K + 1];
    off[0] = 0;
    int least = kMost;                                 // coordinates of the operand with the fewest
    bool broken = false;
#pragma unroll
    for (int t = 0; t < K; ++t) lo[t] = posn0[p * k + (t < k ? t : k - 1)];
#pragma unroll
    for (int t = 0; t < K; ++t) off[t + 1] = posn0[(p + 1) * k + (t < k ? t : k - 1)];
#pragma unroll
    for (int t = 0; t < K; ++t) {
        const int len = t < k ? off[t + 1] - lo[t] : 0;
        broken = broken || len < 0 || len > kMost;
        least = t < k && len < least ? len : least;
        off[t + 1] = off[t] + len;
    }
    // (only operands that violate their preconditions can have more coordinates in a partition than its share)
    broken = broken || off[K] > kRemapGrain + k - 1;
    if (tid == 0) {
        s_fail = 0;
        if (broken) atomicMin(status, (int32_t)NACHO_ERR_INVALID_ARG);
    }
    const int n = broken ? 0 : off[1], all_rows = off[K];
    if (!broken && all_rows > 0) {
        if constexpr (K <= 4) {
            int x[kLoads], q[kLoads];
#pragma unroll
            for (int u = 0; u < kLoads; ++u) {
                const int place = tid + u * kScanThreads;
                // (no branches: places past the last one read it again)
                const int i = place < all_rows ? place : all_rows - 1, j = place < all_rows + k ? place : all_rows + k - 1;
                const int32_t *crd = in.crd0[0], *pos = in.pos1[0];
                int at = lo[0] + i, from = lo[0] + j;
#pragma unroll
                for (int t = 1; t < K; ++t) {
                    crd = i >= off[t] ? in.crd0[t] : crd;
                    at = i >= off[t] ? lo[t] + i - off[t] : at;
                    pos = j >= off[t] + t ? in.pos1[t] : pos;
                    from = j >= off[t] + t ? lo[t] + j - (off[t] + t) : from;
                }
                x[u] = crd[at];
                q[u] = pos[from];
            }
#pragma unroll
            for (int u = 0; u < kLoads; ++u) {
                const int place = tid + u * kScanThreads;
                if (place < all_rows) s_crd[place] = x[u];
                if (place < all_rows + k) s_pos[place] = q[u];
            }
        } else {
            // (many operands, short segments: a place of each at a time)
            int longest = 0;
#pragma unroll
            for (int t = 0; t < K; ++t) longest = off[t + 1] - off[t] > longest ? off[t + 1] - off[t] : longest;
            for (int i = tid; i - tid <= longest; i += kScanThreads) {
                int x[K], q[K];
#pragma unroll
                for (int t = 0; t < K; ++t) {
                    const int len = off[t + 1] - off[t], u = t < k ? t : k - 1;
                    x[t] = in.crd0[u][len > 0 ? lo[t] + (i < len ? i : len - 1) : 0];
                    q[t] = in.pos1[u][lo[t] + (i < len ? i : len)];
                }
#pragma unroll
                for (int t = 0; t < K; ++t) {
                    const int len = off[t + 1] - off[t];
                    if (i < len) s_crd[off[t] + i] = x[t];
                    if (i <= len && t < k) s_pos[off[t] + t + i] = q[t];
                }
            }
        }
    }
    __syncthreads();
    // consecutive rows of operand 0 per thread; the searches of a row in all operands, or of two rows in one, go side by side
    const int each = (n + kScanThreads - 1) / kScanThreads, first = tid * each;
    constexpr int kRows = K == 2 ? 2 : 1;
    int longest = 0;
#pragma unroll
    for (int t = 1; t < K; ++t) longest = off[t + 1] - off[t] > longest ? off[t + 1] - off[t] : longest;
    const int widest = longest > 0 ? 1 << (31 - __builtin_clz((unsigned)longest)) : 0;
    unsigned found = 0u;
    for (int j = 0; j < each; j += kRows) {
        int i[kRows], x[kRows], a[kRows][K];
#pragma unroll
        for (int g = 0; g < kRows; ++g) {
            i[g] = first + j + g < n ? first + j + g : n - 1;
            x[g] = s_crd[i[g]];
#pragma unroll
            for (int t = 1; t < K; ++t) a[g][t] = off[t];      // as many of the segment's rows as lie before x
        }
        for (int step = widest; step > 0; step >>= 1)
#pragma unroll
            for (int t = 1; t < K; ++t)
#pragma unroll
                for (int g = 0; g < kRows; ++g) {
                    const int to = a[g][t] + step, v = s_crd[(to < off[t + 1] ? to : off[t + 1]) - 1];
                    a[g][t] = to <= off[t + 1] && v < x[g] ? to : a[g][t];
                }
#pragma unroll
        for (int g = 0; g < kRows; ++g) {
            bool all = j + g < each && first + j + g < n;
#pragma unroll
            for (int t = 1; t < K; ++t) {
                const int v = s_crd[a[g][t]];
                if (all) s_q[t][i[g]] = (uint16_t)(a[g][t] - off[t]);
                all = all && (t >= k || (a[g][t] < off[t + 1] && v == x[g]));
            }
            found |= all ? 1u << (j + g) : 0u;
        }
    }
    const int mine = __popc(found), incl = wave_inclusive_scan(mine);
    if (lane == NACHO_WAVE - 1) s_count[wave] = incl;
    __syncthreads();
    int m = 0, at = incl - mine;                       // intersected rows of the partition; before this thread's
#pragma unroll
    for (int w = 0; w < kScanWaves; ++w) {
        if (w < wave) at += s_count[w];
        m += s_count[w];
    }
    // Rows without repetitions: every intersected row takes one coordinate of each operand (so they fit s_item, and all
    // partitions together fit the workspace).  Operand 0 repeating a row that the others store breaks that; such a
    // partition contributes nothing.
    if (m > least) {                                   // (uniform)
        m = 0;
        found = 0u;
        if (tid == 0) atomicMin(status, (int32_t)NACHO_ERR_INVALID_ARG);
    }
    for (; found; found &= found - 1u) s_item[at++] = (uint16_t)(first + __ffs(found) - 1);
    __syncthreads();
    // consecutive intersected rows per thread: where their entries start, how many there are
    int start[K][kEach], len[K][kEach], before[K];
#pragma unroll
    for (int t = 0; t < K; ++t)
        if (t < k)
#pragma unroll
            for (int u = 0; u < kEach; ++u) {
                start[t][u] = len[t][u] = 0;
                if (tid * kEach + u < m) {
                    const int i = s_item[tid * kEach + u], q = off[t] + t + (t == 0 ? i : (int)s_q[t][i]);
                    start[t][u] = s_pos[q];
                    len[t][u] = s_pos[q + 1] - start[t][u];
                }
            }
#pragma unroll
    for (int t = 0; t < K; ++t)
        if (t < k) {
            int sum = 0;
#pragma unroll
            for (int u = 0; u < kEach; ++u) sum += len[t][u];
            const int to = wave_inclusive_scan(sum);
            before[t] = to - sum;
            if (lane == NACHO_WAVE - 1) s_len[t][wave] = to;
        }
    __syncthreads();
    // sums along the workgroups: value 0 counts rows, value 1 + t entries of operand t
    auto own = [&](int v) {
        int x = m;
        if (v > 0) {
            x = 0;
#pragma unroll
            for (int w = 0; w < kScanWaves; ++w) x += s_len[v - 1][w];
        }
        return x;
    };
    if (tid <= k && p > 0) publish(state + (int64_t)tid * P0, p, kAggregate, own(tid));
    for (int v = wave; v <= k; v += kScanWaves) {
        int base = 0;
        const bool ok = look_back(state + (int64_t)v * P0, p, own(v), base);
        if (lane == 0) {
            s_base[v] = base;
            if (!ok || (kInstrument && p == in.runs_out)) s_fail = 1;
        }
    }
    __syncthreads();
    const int row0 = s_base[0];
    // (rows past the workspace: only of operands whose rows are not sorted, where partitions can overlap)
    if (s_fail || row0 + m > r.stride) {
        // A workgroup before this one had not published in time.  This one's rows are missing then, whatever the others
        // find (its own counts are published, and the one it waited for may still come), so the kernels after the row loop
        // are told to leave: plan[3] was cleared at the start of the call.
        if (tid == 0) {
            atomicMin(status, (int32_t)(s_fail ? NACHO_ERR_HIP : NACHO_ERR_INVALID_ARG));
            plan[3] = 1;
        }
        return;
    }
#pragma unroll
    for (int u = 0; u < kEach; ++u)
        if (tid * kEach + u < m) r.rows[row0 + tid * kEach + u] = s_crd[s_item[tid * kEach + u]];
#pragma unroll
    for (int t = 0; t < K; ++t)
        if (t < k) {
            int x = s_base[1 + t] + before[t];
#pragma unroll
            for (int w = 0; w < kScanWaves; ++w)
                if (w < wave) x += s_len[t][w];
#pragma unroll
            for (int u = 0; u < kEach; ++u) {
                const int i = row0 + tid * kEach + u;
                if (tid * kEach + u < m) {
                    r.start[(int64_t)t * r.stride + i] = start[t][u];
                    r.cost[(int64_t)t * (r.stride + 1) + i] = x;
                }
                x += len[t][u];
            }
        }
    if (p == P0 - 1 && tid == 0) {                     // the totals
        int64_t total = 0;
        const int rows = row0 + m;
        r.head[0] = rows;
        for (int t = 0; t < k; ++t) {
            const int x = s_base[1 + t] + own(1 + t);
            r.cost[(int64_t)t * (r.stride + 1) + rows] = x;
            r.head[1 + t] = x;
            total += x;
        }
        rule.write(rows, total, plan);
    }
}

// ---- rows of the remapped result that hold an entry --------------------------
constexpr int kKeepItems = 8, kKeepTile = kScanThreads * kKeepItems;

__global__ void __launch_bounds__(kScanThreads)
compact_rows_kernel(const int32_t *__restrict__ rows, const int32_t *__restrict__ pos_full, int most, const int32_t *__restrict__ head,
                    const int64_t *__restrict__ counts_in, const int64_t *__restrict__ plan, SpaddOut out,
                    unsigned long long *__restrict__ state)
{
    __shared__ int s_count[kScanWaves], s_base, s_fail;
    const int tid = threadIdx.x, lane = lane_id(), wave = tid / NACHO_WAVE;
    const int64_t tile = blockIdx.x;
    const int first = (int)tile * kKeepTile + tid * kKeepItems;
    // (the launch is sized for an upper bound of the rows; the loads do not wait for their number: what lies behind is not looked at)
    int x[kKeepItems + 1], row[kKeepItems];
#pragma unroll
    for (int u = 0; u <= kKeepItems; ++u) x[u] = pos_full[first + u < most ? first + u : most];
#pragma unroll
    for (int u = 0; u < kKeepItems; ++u) row[u] = rows[first + u < most ? first + u : most - 1];
    if (plan[3]) return;                               // (the row loop was abandoned)
    const int M = head[0];
    if (tile > 0 && tile * kKeepTile >= M) return;
    unsigned keep = 0u;
#pragma unroll
    for (int u = 0; u < kKeepItems; ++u) keep |= first + u < M && x[u + 1] > x[u] ? 1u << u : 0u;
    const int mine = __popc(keep), incl = wave_inclusive_scan(mine);
    if (lane == NACHO_WAVE - 1) s_count[wave] = incl;
    __syncthreads();
    int own = 0, at = incl - mine;
#pragma unroll
    for (int w = 0; w < kScanWaves; ++w) {
        if (w < wave) at += s_count[w];
        own += s_count[w];
    }
    if (wave == 0) {
        if (lane == 0 && tile > 0) publish(state, tile, kAggregate, own);
        int base = 0;
        const bool ok = look_back(state, tile, own, base);
        if (lane == 0) {
            s_base = base;
            s_fail = ok ? 0 : 1;
        }
    }
    __syncthreads();
    if (s_fail) {
        if (tid == 0) atomicMin(out.status, (int32_t)NACHO_ERR_HIP);
        return;
    }
    at += s_base;
#pragma unroll
    for (int u = 0; u < kKeepItems; ++u)
        if (keep >> u & 1u) {
            if (at < out.cap_rows) {
                out.crd0[at] = row[u];
                out.pos1[at] = x[u];
            }
            ++at;
        }
    if (tid == 0 && (tile + 1) * kKeepTile >= M) {     // the last tile
        const int total = s_base + own;
        const int64_t nnz = counts_in[1];
        out.pos0[0] = 0;
        out.pos0[1] = total;
        if (total <= out.cap_rows) out.pos1[total] = (int32_t)nnz;
        else atomicMin(out.status, (int32_t)NACHO_ERR_CAPACITY);
        out.counts[0] = total;
        out.counts[1] = nnz;
    }
}

__global__ void empty_result_kernel(SpaddOut out, int64_t *info)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        out.pos0[0] = 0;
        out.pos0[1] = 0;
        out.pos1[0] = 0;
        out.counts[0] = 0;
        out.counts[1] = 0;
        *out.status = NACHO_OK;
        info[0] = info[1] = info[2] = info[3] = 0;
    }
}

}  // namespace

int64_t remap_state_words(int64_t P0, int k) { return P0 * (k + 1); }
int64_t compact_state_words(int64_t rows) { return rows > 0 ? (rows + kKeepTile - 1) / kKeepTile : 1; }

hipError_t launch_remap_rows(const DevOperands &ops, int64_t P0, const int32_t *posn0, const RemapArrays &r,
                             unsigned long long *state, int64_t capacity, int64_t round, int64_t P_min, int64_t P_max,
                             int64_t *plan, int32_t *status, hipStream_t s)
{
    RowArrays rows;
    rows.k = ops.k;
    rows.runs_out = nacho_host::wait_runs_out();
    for (int t = 0; t < NACHO_MAX_OPERANDS; ++t) {
        rows.crd0[t] = t < ops.k ? ops.lvl[t][0].crd : nullptr;
        rows.pos1[t] = t < ops.k ? ops.lvl[t][1].pos : nullptr;
    }
    const PlanRule rule = {capacity, round, P_min, P_max};
    auto kernel = ops.k == 2 ? remap_rows_kernel<2> : (ops.k <= 4 ? remap_rows_kernel<4> : (ops.k <= 6 ? remap_rows_kernel<6> : remap_rows_kernel<8>));
    hipLaunchKernelGGL(kernel, dim3((unsigned)P0), dim3(kScanThreads), 0, s, rows, posn0, P0, r, state, rule, plan, status);
    return hipGetLastError();
}

hipError_t launch_compact_rows(const RemapArrays &r, const int32_t *pos_full, const int64_t *counts_in,
                               const int64_t *plan, const SpaddOut &out, unsigned long long *state, hipStream_t s)
{
    // (over the upper bound of the rows; tiles past head[0] leave at once)
    hipLaunchKernelGGL(compact_rows_kernel, dim3((unsigned)compact_state_words(r.stride)), dim3(kScanThreads), 0, s, r.rows,
                       pos_full, (int)r.stride, r.head, counts_in, plan, out, state);
    return hipGetLastError();
}

hipError_t launch_empty_result(const SpaddOut &out, int64_t *info, hipStream_t s)
{
    hipLaunchKernelGGL(empty_result_kernel, dim3(1), dim3(64), 0, s, out, info);
    return hipGetLastError();
}

}  // namespace nacho
