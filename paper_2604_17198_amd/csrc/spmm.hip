// SpMM execution, C = A B with A in CSR and B, C dense row-major: loop order i -> j -> k with the dense k
// innermost (the broadcast rule of Section 4.2.2 scales the cost of every stored non-zero by n, so the
// partitions are those of SpMV), one wavefront per partition.
//
// What bounds it: large matrices the rows of B (30M non-zeros x 256 bytes, 7.7 GB past the L2s at 7 TB/s, unless partitions
// that need the same rows run at the same time on the same XCD: deal_count_kernel below; 1091 to 578 us), all others how many of
// those rows are on their way at a time.  So a row of B is not spread over the whole
// wavefront: a lane takes 16 bytes of it, W = 4 to 16 lanes a row, and the 64 / W groups of lanes of a wavefront each
// walk their own stretch of the partition's non-zeros.  One instruction then asks for up to 16 rows, and the chain of
// dependent steps is that many times shorter (20,000 non-zeros, n = 4: 80 us with a lane per column and the wavefront
// walking all 512 non-zeros of a partition, sixteen at a time).
//
// The wavefront stages crd and val of its partition in LDS and beside every non-zero the row that starts with it, so
// that the walk needs neither pos nor searches and empty rows do not exist for it.  A group keeps the sum of the row
// in hand in registers, stores rows that start and end in its stretch, and keeps the piece in front of its first row
// start (head) and the one of its last row (tail) to the end, where a tail is joined with the heads behind it.  A row
// of C is stored by the partition in which the row starts; the piece of a row that started in an earlier partition
// goes to the carry buffer and is added by the fix-up pass in a fixed order.  No floating-point atomics: results
// repeat bit for bit.
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"

namespace nacho {

namespace {

constexpr int kGrain = 512;                    // most non-zeros of a partition
constexpr int kDealAlone = -1, kDealJoined = -2;       // SpmmDeal::place below 0

// V elements of a row of B or C; in memory they are aligned as one element is (16-byte loads and stores need no more).
template <typename T, int V> struct Piece {
    typedef T type __attribute__((ext_vector_type(V)));
    typedef type mem __attribute__((aligned(sizeof(T))));
};

// W lanes a row, CPL pieces of V elements a lane.  kWhole: there is no partition kernel; the wavefront searches its
// rows, stores its part of the partition table and writes the zeros of its empty rows.
// `deal` (without kWhole): what a workgroup executes, see deal_count_kernel.
// SPMM_SMALL, SPMM_SMALL_DEALT: kWhole for partitions of up to kSmall non-zeros, and those that deal out partitions inside long
// rows by XCD (of SPMM_WHOLE: `deal_rows`).
constexpr int kSmall = 128;
enum SpmmForm { SPMM_TABLE, SPMM_WHOLE, SPMM_SMALL, SPMM_SMALL_DEALT };
template <typename T, int V, int W, int CPL, int kForm>
__global__ void __launch_bounds__(NACHO_WAVE)
spmm_exec_kernel(const int32_t *__restrict__ pos, const int32_t *__restrict__ crd, const T *__restrict__ val,
                 const T *__restrict__ B, int n, int span, int64_t ldb, T *__restrict__ C, int64_t ldc,
                 int32_t *__restrict__ coord, int32_t *__restrict__ posn, int64_t *__restrict__ cost,
                 T *__restrict__ carry_val, int32_t *__restrict__ carry_row, int n_rows, int nnz, int grain,
                 int64_t cost_scale, SpmmDeal deal, bool deal_rows, WaveLog wlog)
{
    constexpr bool kWhole = kForm != SPMM_TABLE, kFew = kForm == SPMM_SMALL || kForm == SPMM_SMALL_DEALT;
    typedef typename Piece<T, V>::type P;
    typedef typename Piece<T, V>::mem PM;
    constexpr int NG = NACHO_WAVE / W;         // groups
    constexpr int kSlots = kGrain + 4 * NG;    // a group's stretch is followed by 4 words (banks of their own for every group)
    constexpr int kIter = (kFew ? kSmall : kGrain) / NACHO_WAVE;
    // non-zeros a group has in flight: 64 registers of B, 16 at most
    constexpr int kRegs = CPL * V * (int)sizeof(T) / 4;
    constexpr int U = kRegs <= 4 ? 16 : (kRegs <= 8 ? 8 : 4);
    const WaveStamp stamp = wave_begin();
    // crd and val; at the end, over them, the heads of the groups
    constexpr int kStaged = kSlots * (4 + (int)sizeof(T)), kHeads = NACHO_WAVE * CPL * (int)sizeof(P);
    __shared__ alignas(16) char smem[kStaged > kHeads ? kStaged : kHeads];
    __shared__ alignas(16) int32_t s_row[kSlots];      // the row that starts with the non-zero, or -1
    T *s_val = reinterpret_cast<T *>(smem);
    int32_t *s_crd = reinterpret_cast<int32_t *>(smem + kSlots * sizeof(T));

    const int lane = threadIdx.x, g = lane / W, gl = lane & (W - 1);
    int p = blockIdx.x, b0 = p, b1 = p + 1;            // b0, b1: the table's boundaries of what is executed
    if (!kWhole && deal.place) {
        const int at = deal.place[p];
        if (at == kDealJoined) {
            if (p >= deal.joined) return;
            b0 = p * deal.join;
            b1 = b0 + deal.join < (int)gridDim.x ? b0 + deal.join : (int)gridDim.x;
        } else if (at >= 0) {
            p = b0 = deal.sorted[at];
            b1 = b0 + 1;
        }
    }
    int r0, r1, n0, n1, len, S, items, base;           // S: a group's stretch, `items` of it non-zeros, from slot `base` on
    int32_t c_in[kIter];
    T v_in[kIter];
    auto stretch = [&]() {
        len = n1 - n0;
        S = ((len + NG - 1) / NG + 3) & ~3;
        const int left = len - g * S;
        items = left < 0 ? 0 : (left < S ? left : S);
        base = g * (S + 4);
    };
    auto stream = [&]() {
        if constexpr (kFew) {
            // (behind the partition's end its last non-zero again, times zero: no branches between the loads)
#pragma unroll
            for (int j = 0; j < kIter; ++j) {
                const int at = g * S + gl + j * W;
                c_in[j] = __builtin_nontemporal_load(crd + (n0 + (at < len ? at : len - 1)));
                v_in[j] = __builtin_nontemporal_load(val + (n0 + (at < len ? at : len - 1)));
            }
            __builtin_amdgcn_sched_barrier(0);
        } else {
#pragma unroll
            for (int j = 0; j < kIter; ++j) {
                const int i = gl + j * W;
                c_in[j] = 0;
                v_in[j] = T(0);
                if (i < items) {
                    c_in[j] = __builtin_nontemporal_load(crd + (n0 + g * S + i));
                    v_in[j] = __builtin_nontemporal_load(val + (n0 + g * S + i));
                }
            }
        }
    };
    // the ends of the first 64 rows, and (kFew) of the first 64 of the rows whose zeros are this wavefront's: all rows are shared out
    // evenly (a large call is bound by what it has in flight: 40M non-zeros, 4 floats, 200 a row 340 us with them, 330 without)
    bool has_head;                                     // row r0 started in an earlier partition
    // (the first row that starts after this partition; unsigned: a lane's row may lie past 2^31)
    unsigned next_first, row;
    int row_a, row_b, zero_a = 0, zero_b = 0;
    const unsigned share = kWhole ? ((unsigned)n_rows + gridDim.x - 1u) / gridDim.x : 0u;
    int z0 = 0, z1 = 0;
    auto rows = [&]() {
        const int pr0 = pos[r0], pr1 = pos[r1];
        row = (unsigned)r0 + (unsigned)lane;
        row_a = row_b = 0;
        if (kWhole) {
            z0 = p * share < (unsigned)n_rows ? (int)(p * share) : n_rows;     // (unsigned: may lie past 2^31)
            z1 = n_rows - z0 < (int)share ? n_rows : z0 + (int)share;
        }
        if constexpr (kFew) {                          // (no branches between the loads)
            const unsigned end = (unsigned)n_rows;
            row_a = pos[row < end ? row : end];
            row_b = pos[row + 1 < end ? row + 1 : end];
            zero_a = pos[z0 + lane < n_rows ? z0 + lane : n_rows];
            zero_b = pos[z0 + lane + 1 < n_rows ? z0 + lane + 1 : n_rows];
        }
        has_head = n0 > pr0;
        next_first = (unsigned)r1 + (n1 > pr1 ? 1u : 0u);
        if constexpr (kFew) {
            if (row >= next_first) row_a = row_b = 0;
        } else {
            if (row < next_first) { row_a = pos[row]; row_b = pos[row + 1]; }
        }
    };
    if (kWhole) {
        // (pos[0] = 0, and every partition has non-zeros)
        const long long Qa = (long long)p * grain, Qb = Qa + grain;
        n0 = (int)(Qa < nnz ? Qa : nnz);
        n1 = (int)(Qb < nnz ? Qb : nnz);
        auto by_rows = [&]() {
            if (r0 >= n_rows) return;
            const int dealt = dealt_partition(p, pos[r0], pos[r0 + 1], grain);
            if (dealt != p) {
                // (a partition inside row r0; it may end with the row)
                p = dealt;
                n0 = p * grain;
                n1 = n0 + grain;
                r1 = r0;
            }
        };
        if constexpr (kFew) {
            // The call is as long as one wavefront's chain of round trips: 64 probes a round instead of 32, and where the non-zeros are known
            // without their rows both are asked for at once (20,000 non-zeros, 37 floats 10.0 to 9.1 us, 100,000, 16 doubles 10.6 to 9.5; with
            // millions of non-zeros the probes' lines cost more than the round: 10M, 4 floats 100 and 114).
            RowWindow wa{0, n_rows}, wb{0, n_rows};
            const int probe = wa.load(pos, n_rows);    // (the first probes are the same for both boundaries)
            if (kForm == SPMM_SMALL) {
                stretch();
                stream();
            }
            wa.narrow(probe, n0);
            wb.narrow(probe, n1);
            while (wa.lo < wa.hi || wb.lo < wb.hi) {
                const int probe_a = wa.load(pos, n_rows), probe_b = wb.load(pos, n_rows);
                wa.narrow(probe_a, n0);
                wb.narrow(probe_b, n1);
            }
            r0 = wa.lo;
            r1 = wb.lo;
        } else rows_holding(pos, n_rows, n0, n1, r0, r1);
        if (p == 0) r0 = 0;
        if (Qb >= nnz) r1 = n_rows;                    // (Qa < nnz)
        if (kForm == SPMM_SMALL_DEALT || (!kFew && deal_rows)) by_rows();
        if (kForm != SPMM_SMALL) {
            stretch();
            stream();
        }
        rows();
    } else {
        r0 = coord[2 * b0]; r1 = coord[2 * b1];
        n0 = posn[2 * b0 + 1]; n1 = posn[2 * b1 + 1];
        stretch();
        stream();
        rows();
    }
    if (kWhole && lane == 0 && blockIdx.y == 0) {
        coord[2 * p] = r0;
        coord[2 * p + 1] = r0 < n_rows && p > 0 ? c_in[0] : 0;
        posn[2 * p] = r0;
        posn[2 * p + 1] = p == 0 ? 0 : (r0 < n_rows ? n0 : nnz);
        cost[p] = (int64_t)n0 * cost_scale;
        if (p == (int)gridDim.x - 1) {
            coord[2 * p + 2] = n_rows;
            coord[2 * p + 3] = 0;
            posn[2 * p + 2] = n_rows;
            posn[2 * p + 3] = nnz;
            cost[p + 1] = (int64_t)nnz * cost_scale;
        }
    }

    // this lane's columns: piece c is at col[c] (the last piece of a row moves back where it would stick out: it holds
    // some columns of the one before it again, with the same sums)
    const int j0 = blockIdx.y * span, width = n - j0 < span ? n - j0 : span;
    const int pieces = (width + V - 1) / V;
    int col[CPL];
    bool mine[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        const int i = c * W + gl;
        mine[c] = i < pieces;
        col[c] = j0 + i * V < n - V ? j0 + i * V : n - V;
    }

#pragma unroll
    for (int j = 0; j < kIter; ++j) {
        const int i = gl + j * W;
        if (i < S) {
            s_crd[base + i] = c_in[j];
            s_val[base + i] = i < items ? v_in[j] : T(0);
            s_row[base + i] = -1;
        }
    }
    unsigned long long empty = kFew ? __ballot(z0 + lane < z1 && zero_a == zero_b) : 0ull;
    wave_sync();
    auto write_zeros = [&]() {
        for (unsigned z = (unsigned)z0; z < (unsigned)z1; z += NACHO_WAVE) {
            if (!kFew || z > (unsigned)z0) empty = __ballot(z + lane < (unsigned)z1 && pos[z + lane] == pos[z + lane + 1]);
            if (empty == 0ull) continue;
            for (int i = g; i < NACHO_WAVE; i += NG)
                if (bit_at(empty, i)) {
#pragma unroll
                    for (int c = 0; c < CPL; ++c)
                        if (mine[c]) *reinterpret_cast<PM *>(C + (int64_t)(z + i) * ldc + col[c]) = P(T(0));
                }
        }
    };
    // (a small call's chain goes first; a large one has other wavefronts: at the end 2M non-zeros, 4 floats take 27.7 us, here 26.5)
    if (kWhole && !kFew) write_zeros();
    const float per_S = 1.0f / (float)S;
    for (;;) {                                         // rows, 64 at a time
        const bool is_row = row < next_first;
        if (is_row && row_b > row_a && row_a >= n0) {
            const int i = row_a - n0;                  // (< len: the row starts in this partition)
            const int at = (int)(((float)i + 0.5f) * per_S);       // i / S
            s_row[i + 4 * at] = (int)row;
        }
        const unsigned next = (unsigned)__builtin_amdgcn_readfirstlane((int)row) + NACHO_WAVE;
        if (next >= next_first) break;
        unsigned from = next;
        if (__ballot(row_b > row_a) == 0ull) {
            // 64 rows without an entry: however many there are, stepped over
            const int q = __builtin_amdgcn_readfirstlane(row_b);
            if (q >= n1) break;
            from = (unsigned)first_row_past(pos, (int)next, (int)next_first, q);
        }
        row = from + lane;
        row_a = row_b = 0;
        if (row < next_first) { row_a = pos[row]; row_b = pos[row + 1]; }
    }
    wave_sync();

    P acc[CPL], head[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) acc[c] = head[c] = P(T(0));
    int cur = -1;                                      // the row in hand; -1: one that started before the stretch
    auto store_row = [&](int r, const P (&x)[CPL]) {
#pragma unroll
        for (int c = 0; c < CPL; ++c)
            if (mine[c]) *reinterpret_cast<PM *>(C + (int64_t)r * ldc + col[c]) = x[c];
    };
    // N non-zeros from slot base + i0 on; kAll: all of them lie in the stretch
    auto step = [&](int i0, auto count, auto all) {
        constexpr int N = decltype(count)::value;
        constexpr bool kAll = decltype(all)::value;
        P b[N][CPL];
        int r[N];
        T v[N];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int64_t at = (int64_t)s_crd[base + i0 + u] * ldb;
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                b[u][c] = P(T(0));
                if (mine[c] && (kAll || i0 + u < items)) b[u][c] = *reinterpret_cast<const PM *>(B + at + col[c]);
            }
        }
#pragma unroll
        for (int u = 0; u < N; ++u) {
            r[u] = s_row[base + i0 + u];
            v[u] = s_val[base + i0 + u];
        }
#pragma unroll
        for (int u = 0; u < N; ++u) {
            if (r[u] >= 0) {
                if (cur >= 0) store_row(cur, acc);
                else {
#pragma unroll
                    for (int c = 0; c < CPL; ++c) head[c] = acc[c];
                }
#pragma unroll
                for (int c = 0; c < CPL; ++c) acc[c] = P(T(0));
                cur = r[u];
            }
#pragma unroll
            for (int c = 0; c < CPL; ++c) acc[c] += v[u] * b[u][c];
        }
    };
    int i0 = 0;
    for (; i0 + U <= items; i0 += U) step(i0, std::integral_constant<int, U>(), std::true_type());
    for (; i0 < items; i0 += 4) step(i0, std::integral_constant<int, 4>(), std::false_type());
    if (cur < 0) {
#pragma unroll
        for (int c = 0; c < CPL; ++c) head[c] = acc[c];
    }

    // a group's last row goes on in the heads of the groups behind it, up to the first that starts a row of its own
    const unsigned long long started = __ballot(cur >= 0);
    wave_sync();
    P *s_head = reinterpret_cast<P *>(smem);
#pragma unroll
    for (int c = 0; c < CPL; ++c) s_head[c * NACHO_WAVE + lane] = head[c];
    wave_sync();
    auto starts = [&](int h) { return bit_at(started, h * W); };
    auto add_heads = [&](P (&x)[CPL]) {
        for (int h = g + 1; h < NG; ++h) {
#pragma unroll
            for (int c = 0; c < CPL; ++c) x[c] += s_head[c * NACHO_WAVE + h * W + gl];
            if (starts(h)) break;
        }
    };
    if (cur >= 0) {
        add_heads(acc);
        store_row(cur, acc);
    }
    if (has_head && g == 0) {                          // the piece of the row that started in an earlier partition
        if (cur < 0) add_heads(head);
#pragma unroll
        for (int c = 0; c < CPL; ++c)
            if (mine[c]) *reinterpret_cast<PM *>(carry_val + (int64_t)p * n + col[c]) = head[c];
    }
    if (lane == 0 && blockIdx.y == 0) carry_row[p] = has_head ? r0 : -1;
    if (kFew) write_zeros();
    if (blockIdx.y == 0) wave_end(wlog, p, stamp, (uint32_t)len, (uint32_t)(next_first - r0));
}

// Carry fix-up: 64 / V lanes per partition, a piece of V columns each: 16 partitions (floats), 8 (doubles) or 4 (fewer columns
// than a 16-byte piece has) per workgroup.  The carries of a row lie in consecutive partitions; the lanes of the first one add the
// run to the row of C.  A run of more than kShort carries (there is at most one per workgroup: it is longer than the workgroup's
// partitions) is added by the whole workgroup, every group an equal share of it: the largest row of 30M non-zeros has a thousand,
// which one wavefront, a row of carries at a time, took 35 us for (half as many).  The order of the additions is fixed.
// What bounds it: round trips, of which there are two: the rows of the carries and the first of each, then the rows of C.  (Where the
// run ends was looked up in the matrix, in front of the carries: 156k partitions of 64 floats 26.8 us, so 20.9; calls of 100k
// non-zeros 9.6, so 9.0.)  Loads are as wide as the lanes' pieces.
constexpr int kFixCols = 64, kShort = 32;

template <typename T, int V>
__global__ void __launch_bounds__(256)
spmm_fixup_kernel(T *__restrict__ C, int64_t ldc, int n, int P, const T *__restrict__ carry_val,
                  const int32_t *__restrict__ carry_row, const int32_t *__restrict__ pos,
                  const int32_t *__restrict__ posn, int grain, SpmmDeal deal)
{
    typedef typename Piece<T, V>::type Vec;
    typedef typename Piece<T, V>::mem Mem;
    constexpr int kFixLanes = kFixCols / V, kFixGroups = 256 / kFixLanes;
    static_assert(kShort >= kFixGroups, "one long run per workgroup");
    static_assert(kFixGroups + kShort < NACHO_WAVE && kShort == 32, "a lane for every carry that is looked at");
    __shared__ Vec part[kFixGroups][kFixLanes];
    const int g = threadIdx.x / kFixLanes, gl = threadIdx.x & (kFixLanes - 1), lane = lane_id();
    const int p0 = blockIdx.x * kFixGroups, p = p0 + g;
    // (n >= V; the last piece of a row moves back where it would stick out: the columns it shares with the one before are
    // that one's to store)
    const int j0 = blockIdx.y * (kFixLanes * V) + gl * V, col = j0 < n - V ? j0 : n - V, shared = j0 - col;
    // In one trip to memory: the rows of the carries, from the one before the workgroup's first on, a lane each (every wavefront for
    // itself); the first carry of every group's run, if it starts one; whether partitions were joined.  Places past the last
    // partition read that one.
    const int seen = p0 - 1 + lane;
    int row = carry_row[seen < 0 ? 0 : (seen < P ? seen : P - 1)];
    const Vec own = *reinterpret_cast<const Mem *>(carry_val + (int64_t)(p < P ? p : P - 1) * n + col);
    const int place = *(deal.join > 1 ? deal.place + p0 : carry_row + p0);
    if (deal.join > 1 && place == kDealJoined) {
        // (a carry for every `join` partitions; place is the same throughout then)
        P = deal.joined;
        grain *= deal.join;
        if (p0 >= P) return;
    }
    row = seen >= 0 && seen < P ? row : -1;
    const int left = lane_left(row);                   // (with all lanes on)
    const unsigned long long on = __ballot(row >= 0 && row == left && lane > 0);       // goes on with the row before it
    const unsigned long long starts = __ballot(row >= 0) & ~on;
    // carries of the row of place `at`, as far as they are looked at; workgroups have groups in places 1 to kFixGroups
    auto run_from = [&](int at) {
        const unsigned behind = __builtin_amdgcn_alignbit((unsigned)(on >> 32), (unsigned)on, at + 1);     // kShort of them
        return behind == ~0u ? kShort + 1 : __ffs(~behind);
    };
    const unsigned long long longer = __ballot(lane > 0 && lane <= kFixGroups && bit_at(starts, lane) && run_from(lane) > kShort);
    const int run = run_from(g + 1), r = value_from(row, g + 1);
    const bool first = bit_at(starts, g + 1);
    // carries q, q + step, ... below `to`, eight 16-byte pieces or sixteen narrower ones in flight
    auto sum = [&](int q, int to, int step) -> Vec {
        Vec x = Vec(T(0));
        constexpr int kFlight = sizeof(Vec) == 16 ? 8 : 16;
        for (; q < to; q += kFlight * step) {
            Vec t[kFlight];
#pragma unroll
            for (int u = 0; u < kFlight; ++u) {
                t[u] = Vec(T(0));
                if (q + u * step < to) t[u] = *reinterpret_cast<const Mem *>(carry_val + (int64_t)(q + u * step) * n + col);
            }
#pragma unroll
            for (int u = 0; u < kFlight; ++u) x += t[u];
        }
        return x;
    };
    const bool mine = j0 < n;
    T *const at = C + (int64_t)r * ldc + col;          // (used by the first of a run)
    auto put = [&](T *to, Vec x) {
        if (shared == 0) *reinterpret_cast<Mem *>(to) = x;
        else
#pragma unroll
            for (int c = 1; c < V; ++c)
                if (c >= shared) to[c] = x[c];
    };
    if (first && run <= kShort) {
        if (mine) {
            const Vec y = *reinterpret_cast<const Mem *>(at);
            put(at, y + (own + sum(p + 1, p + run, 1)));
        }
    }
    if (longer == 0ull) return;                        // (the whole workgroup)
    // the run ends with the last partition that starts inside the row
    const int at_long = __ffsll((long long)longer) - 1, first_long = p0 + at_long - 1, row_long = lane_value(row, at_long);
    const int row_end = pos[row_long + 1];
    int end_long = P;
    if (grain > 0) end_long = shares_before(row_end, grain);           // (pos[0] = 0)
    else {
        int lo = first_long + 1, hi = P;               // the first partition that starts at or behind the row's end
        while (lo < hi) {
            const int mid = lo + ((hi - lo) >> 1);
            if (posn[2 * mid + 1] < row_end) lo = mid + 1; else hi = mid;
        }
        end_long = lo;
    }
    end_long = end_long < P ? end_long : P;
    part[g][gl] = mine ? sum(first_long + g, end_long, kFixGroups) : Vec(T(0));
    __syncthreads();
    if (g == 0 && mine) {
        Vec y = Vec(T(0));
#pragma unroll
        for (int u = 0; u < kFixGroups; ++u) y += part[u][gl];
        T *const to = C + (int64_t)row_long * ldc + col;
        put(to, *reinterpret_cast<const Mem *>(to) + y);
    }
}

// ---- which workgroup executes which partition ----------------------------------
// The rows of B that the partitions of long rows gather ascend with the partition: a partition inside a row covers a
// stretch of columns, and so do those of every other long row.  Executed in the order of their columns, partitions that need the same
// rows of B run at the same time, and dealt out so that an XCD gets one eighth of the columns they find them in its L2.  (A
// workgroup runs on XCD index mod 8, and workgroups start in the order of their indexes.)  So the partitions that lie
// inside one row are sorted by their first column, the sorted list is cut into eight stretches, one for the workgroups of
// every residue, and those workgroups take their stretch in order.  All other partitions stay where they are: they miss the
// L2 whatever their order, and the memory system and the L2s work at the same time.
// A counting sort in two kernels: counts per workgroup and bin, then places.  The order inside a bin is left to chance;
// nothing that is computed hangs on it.
//
// Partitions of 64 or 128 non-zeros write and add four to eight times the carries of 512, which pays where neighbours share rows of B,
// sorted or as they are.  Where they do not, a wavefront executes `join` partitions of the table in one piece, as long as an unsorted
// call's: where fewer than 1/8 of the partitions lie inside a row and cover less than a third of the columns (rows of 100, 6M
// non-zeros, 200 doubles, columns at random: whatever they cover 1515 us, half 1508, a third 1390; rows of 300: 746, 746, 775),
// and the first columns of fewer than half of the neighbours are within 4 MB of B (an L2) and an eighth of the columns of each
// other.  (6M non-zeros, 200 doubles, us, each partition alone and joined: rows of 30 with columns at random 1639 and 1521, in a
// band of 4000 columns 836 and 1389; rows by Zipf's law, 30 on average, 860 and 1527.)
constexpr int kDealGroups = 32, kDealBins = 512, kDealThreads = 1024, kDealWords = kDealBins + 9;

// Of the lanes with the same residue (mod 8): how many are set in `mask`, and how many of those below this lane.
__device__ inline int class_count(unsigned long long mask, int residue)
{
    const unsigned mine = 0x01010101u << residue;
    return __popc((unsigned)mask & mine) + __popc((unsigned)(mask >> 32) & mine);
}
__device__ inline int class_rank(unsigned long long mask, int residue)
{
    const unsigned mine = 0x01010101u << residue;
    return __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32) & mine, __builtin_amdgcn_mbcnt_lo((unsigned)mask & mine, 0u));
}

// place[p]: the bin of a partition inside one row, else -1.  counts: of the bins, of the residues, of neighbours near each other.
__global__ void __launch_bounds__(kDealThreads)
deal_count_kernel(const int32_t *__restrict__ coord, int P, int chunk, int shift, int most_span, int near_columns,
                  int32_t *__restrict__ place, int32_t *__restrict__ counts)
{
    __shared__ int s_count[kDealWords];
    if (threadIdx.x < kDealWords) s_count[threadIdx.x] = 0;
    __syncthreads();
    const int lane = lane_id();
    const int first = blockIdx.x * chunk, end = P < first + chunk ? P : first + chunk;
    for (int p0 = first + (int)threadIdx.x - lane; p0 < end; p0 += kDealThreads) {
        const int p = p0 + lane;
        int bin = -1;
        bool near = false;
        if (p < end) {
            const int2 *boundary = reinterpret_cast<const int2 *>(coord) + p;
            const int2 a = boundary[0], e = boundary[1];       // row and column
            // (a partition inside one row: its end lies in the row it starts in; one that covers more columns is nobody's neighbour)
            if (a.x == e.x && e.y - a.y <= most_span) bin = (a.y >> shift) & (kDealBins - 1);
            near = abs(e.y - a.y) <= near_columns;
            place[p] = bin;
        }
        if (bin >= 0) atomicAdd(&s_count[bin], 1);
        const unsigned long long inside = __ballot(bin >= 0);
        if (lane < 8 && inside) atomicAdd(&s_count[kDealBins + lane], class_count(inside, lane));       // (p0: a multiple of 64)
        const unsigned long long close = __ballot(near);
        if (lane == 8) atomicAdd(&s_count[kDealBins + 8], __popcll(close));
    }
    __syncthreads();
    if (threadIdx.x < kDealWords) counts[blockIdx.x * kDealWords + threadIdx.x] = s_count[threadIdx.x];
}

__global__ void __launch_bounds__(kDealThreads)
deal_place_kernel(int P, int chunk, const int32_t *__restrict__ counts, SpmmDeal deal)
{
    __shared__ int s_at[kDealWords], s_wave[kDealThreads / NACHO_WAVE], s_class[9];
    const int tid = threadIdx.x, lane = lane_id(), wave = tid / NACHO_WAVE;
    // a thread per count: of all workgroups, and of those before this one
    int all = 0, before = 0;
    if (tid < kDealWords) {
        int c[kDealGroups];
#pragma unroll
        for (int u = 0; u < kDealGroups; ++u) c[u] = counts[u * kDealWords + tid];
#pragma unroll
        for (int u = 0; u < kDealGroups; ++u) {
            all += c[u];
            before += u < (int)blockIdx.x ? c[u] : 0;
        }
    }
    const int incl = wave_inclusive_scan(all);
    if (lane == NACHO_WAVE - 1) s_wave[wave] = incl;
    if (tid >= kDealBins && tid < kDealWords) s_class[tid - kDealBins] = all;
    __syncthreads();
    int inside = 0;
    for (int u = 0; u < 8; ++u) inside += s_class[u];
    const bool joined = deal.join > 1 && inside < P / 8 && s_class[8] < P / 2;
    if (tid < kDealBins) {
        int base = incl - all;
        for (int u = 0; u < wave; ++u) base += s_wave[u];
        s_at[tid] = base + before;
    } else if (tid < kDealBins + 8) {
        int start = 0;
        for (int u = 0; u < tid - kDealBins; ++u) start += s_class[u];
        s_at[tid] = start + before;
    }
    __syncthreads();
    const int first = blockIdx.x * chunk, end = P < first + chunk ? P : first + chunk;
    if (joined) {
        for (int p = first + tid; p < end; p += kDealThreads) deal.place[p] = kDealJoined;
        return;
    }
    for (int p0 = first + tid - lane; p0 < end; p0 += kDealThreads) {
        const int p = p0 + lane, residue = lane & 7;           // (p0: a multiple of 64)
        const int bin = p < end ? deal.place[p] : -1;
        const unsigned long long mask = __ballot(bin >= 0);
        int at = 0;
        if (lane < 8) at = atomicAdd(&s_at[kDealBins + residue], class_count(mask, residue));
        at = __shfl(at, residue, NACHO_WAVE) + class_rank(mask, residue);
        if (bin >= 0) deal.sorted[atomicAdd(&s_at[bin], 1)] = p;
        if (p < end) deal.place[p] = bin >= 0 ? at : kDealAlone;
    }
}

}  // namespace

int64_t spmm_deal_words(int64_t P) { return 2 * P + kDealGroups * kDealWords; }

hipError_t launch_spmm_deal(const int32_t *coord, int64_t P, int64_t n_cols, int64_t row_bytes, int join, int32_t *words,
                            SpmmDeal *deal, hipStream_t stream)
{
    int shift = 0;
    while ((n_cols - 1) >> shift >= kDealBins) ++shift;
    const int chunk = (int)((P + kDealGroups * NACHO_WAVE - 1) / (kDealGroups * NACHO_WAVE)) * NACHO_WAVE;
    const int near_columns = (int)(4000000 / row_bytes < n_cols / 8 ? 4000000 / row_bytes : n_cols / 8);
    int32_t *counts = words;
    deal->place = counts + kDealGroups * kDealWords;
    deal->sorted = deal->place + P;
    deal->join = join;
    deal->joined = (int)((P + join - 1) / join);
    hipLaunchKernelGGL(deal_count_kernel, dim3(kDealGroups), dim3(kDealThreads), 0, stream, coord, (int)P, chunk, shift,
                       (int)(n_cols / 3), near_columns, deal->place, counts);
    hipLaunchKernelGGL(deal_place_kernel, dim3(kDealGroups), dim3(kDealThreads), 0, stream, (int)P, chunk, counts, *deal);
    return hipGetLastError();
}

int spmm_capacity() { return kGrain; }

// Non-zeros per partition when the caller leaves the partitioning to the library: enough wavefronts for the chip.
// Calls that sort their partitions take shorter ones, which cover fewer columns, the shorter the wider a row of B is: its
// gathers are what that saves, the carries what it costs (10M non-zeros in 200k rows, 256, 192, 128 and 64 non-zeros, us: 16
// floats 105, 111, 125, -; 64 198, 194, 195, 237; 64 doubles 429, 404, 380, 374; 200 doubles 1635, 1532, 1397, 1284).
int spmm_grain(int64_t nnz, int units, bool dealt, int64_t row_bytes)
{
    if (dealt) return row_bytes >= 768 ? 64 : (row_bytes >= 384 ? 128 : (row_bytes >= 144 ? 192 : 256));
    const int64_t per = nnz / ((int64_t)units * 16);
    return per >= kGrain ? kGrain : (per < 64 ? 64 : (int)((per + 63) / 64 * 64));
}

// Whether a call sorts its partitions: the partition kernel and the two of the sort are 14 us (24 with 150k partitions), which pays
// from about 600 MB of gathers on, at least a cache line each (us, unsorted and sorted, rows by Zipf's law, 30 on average: 400k
// non-zeros, 200 doubles 71 and 66; 1M, 200 floats 105 and 80; 3M, 64 floats 92 and 72; 5M, 32 floats 76 and 69), while B is
// larger than an L2 where its rows are shorter than a line (10M non-zeros, 16 floats, 5 MB of B 117 and 100; 4 doubles: 5M,
// 3.2 MB 63 and 65), than two L2s for others (Zipf's law, 1.2; B of 7, 9, 11 and 14 MB; 8M, 32 floats 87 and 90, 90 and 92, 93 and
// 92, 100 and 95; 6M, 64 floats 98 and 104, 110 and 106, 124 and 108, 137 and 113; 2M, 200 floats 118 and 120, 138 and 123, 153
// and 124, 166 and 126; 1M, 200 doubles 98 and 115, 107 and 116, 117 and 119, 133 and 121).  What this costs matrices of short rows
// with columns at random, which have nothing to sort: 1 to 8 % of such calls, 10 to 15 % of the smallest (1.3M, 64 doubles, rows of
// 20: 92 and 105).
bool spmm_dealt(int64_t nnz, int64_t n_cols, int64_t row_bytes)
{
    return (double)nnz * (double)(row_bytes > 128 ? row_bytes : 128) >= 6e8 &&
           (double)n_cols * (double)row_bytes >= (row_bytes >= 256 ? 9e6 : (row_bytes >= 128 ? 7.8e6 : 4e6));
}

// Fixed-grain calls do without a partition kernel: the wavefronts of the executing kernel find their rows in two to
// four rounds of loads, which hide behind each other, and its place in the stream is saved (100k non-zeros, 16 floats:
// 12.8 to 10.4 us; 2M, 16 floats: 37.7 to 33.7; 30M, 4 floats: 353 to 332).  The zeros of empty rows are spread over the
// wavefronts; where that would be thousands of rows each, the partition kernel writes them.
bool spmm_whole(int64_t P, int64_t n_rows) { return n_rows <= P * 1024; }

hipError_t launch_spmm_exec(int dtype, const int32_t *pos, const int32_t *crd, const void *val,
                            const void *B, int n, int64_t ldb, void *C, int64_t ldc, int64_t n_rows, int64_t nnz,
                            int32_t *coord, int32_t *posn, int64_t *cost, int64_t P, void *carry_val,
                            int32_t *carry_row, int64_t grain, int64_t cost_scale, bool whole, const SpmmDeal &deal,
                            double b_bytes, hipStream_t stream)
{
    const int V = dtype == NACHO_F64 ? 2 : 4;
    // (an L2 holds 4 MB; 1.3M non-zeros, 37 columns of doubles, 15 MB of B: 65 to 48 us)
    const bool deal_rows = b_bytes > 4e6;
    const int form = !whole ? SPMM_TABLE : (grain > kSmall ? SPMM_WHOLE : (deal_rows ? SPMM_SMALL_DEALT : SPMM_SMALL));
    // stretches of up to 64 pieces of V columns, of about equal width
    const int pieces = n < V ? n : (n + V - 1) / V, stretches = (pieces + NACHO_WAVE - 1) / NACHO_WAVE;
    const int per = (pieces + stretches - 1) / stretches;
    const int span = n < V ? n : per * V;
#define NACHO_SPMM_LAUNCH(T, VV, W, CPL, WHOLE)                                                                         \
    hipLaunchKernelGGL((spmm_exec_kernel<T, VV, W, CPL, WHOLE>), dim3((unsigned)P, (unsigned)stretches), dim3(NACHO_WAVE), 0,  \
                       stream, pos, crd, (const T *)val, (const T *)B, n, span, ldb, (T *)C, ldc, coord, posn, cost,    \
                       (T *)carry_val, carry_row, (int)n_rows, (int)nnz, (int)grain, cost_scale, deal, deal_rows, \
                       nacho_host::wave_log())
#define NACHO_SPMM_SHAPE(T, VV, W, CPL)                                                                                 \
    do {                                                                                                                \
        if (form == SPMM_WHOLE) NACHO_SPMM_LAUNCH(T, VV, W, CPL, SPMM_WHOLE);                                           \
        else if (form == SPMM_SMALL) NACHO_SPMM_LAUNCH(T, VV, W, CPL, SPMM_SMALL);                                      \
        else if (form == SPMM_SMALL_DEALT) NACHO_SPMM_LAUNCH(T, VV, W, CPL, SPMM_SMALL_DEALT);                          \
        else NACHO_SPMM_LAUNCH(T, VV, W, CPL, SPMM_TABLE);                                                              \
    } while (0)
    // the fewest lanes that hold a row: more rows in flight per instruction
#define NACHO_SPMM_TYPE(T, VV)                                                                                          \
    do {                                                                                                                \
        if (n < VV) NACHO_SPMM_SHAPE(T, 1, 4, 1);                                                                       \
        else if (per <= 4) NACHO_SPMM_SHAPE(T, VV, 4, 1);                                                               \
        else if (per <= 8) NACHO_SPMM_SHAPE(T, VV, 8, 1);                                                               \
        else if (per <= 16) NACHO_SPMM_SHAPE(T, VV, 16, 1);                                                             \
        else if (per <= 32) NACHO_SPMM_SHAPE(T, VV, 16, 2);                                                             \
        else if (per <= 48) NACHO_SPMM_SHAPE(T, VV, 16, 3);                                                             \
        else NACHO_SPMM_SHAPE(T, VV, 16, 4);                                                                            \
    } while (0)
    if (dtype == NACHO_F64) NACHO_SPMM_TYPE(double, 2);
    else NACHO_SPMM_TYPE(float, 4);
#undef NACHO_SPMM_TYPE
#undef NACHO_SPMM_SHAPE
#undef NACHO_SPMM_LAUNCH
    return hipGetLastError();
}

hipError_t launch_spmm_fixup(int dtype, void *C, int64_t ldc, int n, int64_t P, const void *carry_val,
                             const int32_t *carry_row, const int32_t *pos, const int32_t *posn, int64_t grain,
                             const SpmmDeal &deal, hipStream_t stream)
{
#define NACHO_FIXUP_LAUNCH(T, V)                                                                                        \
    hipLaunchKernelGGL((spmm_fixup_kernel<T, V>),                                                                       \
                       dim3((unsigned)((P * (kFixCols / V) + 255) / 256), (unsigned)((n + kFixCols - 1) / kFixCols)),   \
                       dim3(256), 0, stream, (T *)C, ldc, n, (int)P, (const T *)carry_val, carry_row, pos, posn, (int)grain, deal)
    if (dtype == NACHO_F64) {
        if (n >= 2) NACHO_FIXUP_LAUNCH(double, 2);
        else NACHO_FIXUP_LAUNCH(double, 1);
    } else {
        if (n >= 4) NACHO_FIXUP_LAUNCH(float, 4);
        else NACHO_FIXUP_LAUNCH(float, 1);
    }
#undef NACHO_FIXUP_LAUNCH
    return hipGetLastError();
}

}  // namespace nacho
