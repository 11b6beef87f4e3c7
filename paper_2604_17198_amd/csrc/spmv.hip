// SpMV execution: one wavefront per partition (the compute kernel of Section
// 4.4 with loop bounds taken from the stored partitions), plus the carry
// fix-up for rows split across partitions.
//
// Partition p owns the stored non-zeros at positions [n_p, n_{p+1}) of A.  Its
// wavefront
//   1. streams crd/val of that range (read once: non-temporal loads, so that
//      the L2 is left to x), gathers x and leaves the products in LDS;
//   2. walks the rows that overlap the range (their pos entries staged in LDS),
//      one lane per row; rows with many products are summed by the whole
//      wavefront instead;
//   3. stores y[r] for every row that STARTS inside the partition (a row that
//      ends later gets its first piece here), and hands the piece of the one
//      row that started earlier to the fix-up pass as a carry.
// The fix-up pass adds the carries of a row, in a fixed order, to y[r].  There
// are no floating-point atomics anywhere: results repeat bit for bit.
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"

namespace nacho {

namespace {

// Products per row from which the wavefront sums it together.  Below, the row's lane does, four products at a time:
// the wavefront takes as long as its longest such row, a round trip to LDS per step (40,000 non-zeros, where nothing
// else hides it: 13.5 us with one product at a time and rows of up to 191 of them, 5 us like this).
constexpr int kLongRow = 48;

// Rows whose zeros one wavefront of a call without a partition kernel may have to write: one batch of loads.
constexpr int kZeroRows = 256;

// kDealt: the partitions come from fixed-grain queries (grain > 0) and are dealt out by XCD; the
// instantiation without it serves arbitrary partition tables (caller's P, the row-aware cost).
// kFused (with kDealt): there is no partition table; the wavefront finds its own two boundaries, the
// search of Algorithm 1 for one CSR operand (Section 4.2.2: the row with pos[r] <= Q < pos[r + 1], at
// position Q) with the fixed-grain queries Q_b = min(b * grain, nnz), as a 64-ary search over pos.
// kTable (with kFused): the wavefront stores its boundary in the partition table, and the zeros of empty rows, wherever
// they lie, are shared out evenly over the wavefronts (at most kZeroRows rows each).
template <typename T, int G, int RBLK, bool kDealt, bool kFused = false, bool kTable = false>
__global__ void __launch_bounds__(NACHO_WAVE)
spmv_exec_kernel(const int32_t *__restrict__ pos, const int32_t *__restrict__ crd,
                 const T *__restrict__ val, const T *__restrict__ x, T *__restrict__ y,
                 int nnz, int32_t *__restrict__ coord, int32_t *__restrict__ posn, int64_t *__restrict__ cost,
                 T *__restrict__ carry_val, int32_t *__restrict__ carry_row, int n_rows, int grain, WaveLog wlog)
{
    const WaveStamp stamp = wave_begin();
    __shared__ T prod[G + 8];
    __shared__ int32_t spos[RBLK + 1];

    const int lane = threadIdx.x;
    // What bounds a small or middling call is the chain of round trips of one wavefront, so nothing waits that does not have to:
    // where partitions have a fixed grain their non-zeros are known without their rows, and crd / val travel beside the search for
    // the rows or the table's row fields, the gathers of x beside its later rounds, the rows' positions beside the gathers (the
    // search, the row positions and then the non-zeros one after the other 40,000 non-zeros of doubles took 9.9 us, 5M floats of 50 a row
    // 29.6, 20M of 12 a row 112, like this 8.2, 25.5 and 107).
    int p = blockIdx.x;
    int r0 = 0, r1 = 0, n0 = 0, n1 = 0;                // rows and positions of the boundaries p and p + 1
    auto fixed_range = [&]() {
        const long long Qa = (long long)p * grain, Qb = Qa + grain;
        n0 = (int)(Qa < nnz ? Qa : nnz);               // (pos[0] = 0)
        n1 = (int)(Qb < nnz ? Qb : nnz);
    };
    auto ends = [&]() {                                // of the table: by definition
        if (p == 0) r0 = 0;
        else if ((long long)p * grain >= nnz) r0 = n_rows;
        if ((long long)(p + 1) * grain >= nnz) r1 = n_rows;
    };
    RowWindow wa, wb;                                  // (kTable) the rows that hold n0 and n1
    int probe = 0;
    if (kTable) {
        wa = wb = RowWindow{0, n_rows};
        probe = wa.load(pos, n_rows);                  // (the first probes are the same for every boundary)
        fixed_range();
    } else if (kFused) {
        fixed_range();
        rows_holding(pos, n_rows, n0, n1, r0, r1);
        ends();
    }
    // Which partition this workgroup executes: those inside one long row are dealt out by XCD, so that the gathers of an XCD
    // stay inside one eighth of x, which its L2 holds (all of x it does not).
    // (k = 1, d = 2: coord[b*2 + 0] = row, posn[b*2 + 1] = position in crd/val)
    if (kDealt) {
        const int r = kFused ? r0 : coord[2 * p];
        if (r < n_rows) p = dealt_partition(p, pos[r], pos[r + 1], grain);
        if (!kFused || p != (int)blockIdx.x) fixed_range();
        if (kFused && p != (int)blockIdx.x) {
            rows_holding(pos, n_rows, n0, n1, r0, r1);
            ends();
        }
    }
    if (!kFused) {
        r0 = coord[2 * p]; r1 = coord[2 * p + 2];
        if (!kDealt) { n0 = posn[2 * p + 1]; n1 = posn[2 * p + 3]; }
    }
    const int a0 = n0;                                 // prod[i] belongs to position a0 + i

    // Lane l takes positions n0 + l, n0 + 64 + l, ...: consecutive lanes hold
    // consecutive non-zeros, so inside a dense row the 64 gathers of one
    // instruction fall into few cache lines of x (columns are sorted).  All
    // streamed loads are issued before the first gather, all gathers before the
    // first LDS store, so one wavefront keeps its whole window in flight.
    // (what lies past the partition's last place is loaded from that place, and nobody's product)
    constexpr int kIter = G / NACHO_WAVE;
    const int last = n1 - n0 - 1;                      // (kTable: every partition has non-zeros)
    int c[kIter];
    T v[kIter], xv[kIter];
    if (kTable || last >= 0) {
#pragma unroll
        for (int j = 0; j < kIter; ++j) {
            const int i = j * NACHO_WAVE + lane;
            c[j] = __builtin_nontemporal_load(crd + n0 + (i < last ? i : last));
        }
#pragma unroll
        for (int j = 0; j < kIter; ++j) {
            const int i = j * NACHO_WAVE + lane;
            v[j] = __builtin_nontemporal_load(val + n0 + (i < last ? i : last));
        }
        __builtin_amdgcn_sched_barrier(0);             // (left to itself the compiler asks for val behind the gathers)
    }
    if (kTable) {
        wb.narrow(probe, n1);
        wa.narrow(probe, n0);
        const int probe_a = wa.load(pos, n_rows), probe_b = wb.load(pos, n_rows);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < kIter; ++j) asm volatile("" : "+v"(c[j]));         // (nor does anything of the gathers' wait before this)
#pragma unroll
        for (int j = 0; j < kIter; ++j) xv[j] = x[c[j]];
        __builtin_amdgcn_sched_barrier(0);
        wa.narrow(probe_a, n0);
        wb.narrow(probe_b, n1);
        while (wa.lo < wa.hi || wb.lo < wb.hi) {
            const int more_a = wa.load(pos, n_rows), more_b = wb.load(pos, n_rows);
            wa.narrow(more_a, n0);
            wb.narrow(more_b, n1);
        }
        r0 = wa.lo;
        r1 = wb.lo;
        ends();
    }
    // the positions of the first row block: one lane a row, the first kAhead * 64 of them through registers, so that neither the
    // gathers wait for them nor they for the gathers
    constexpr int kAhead = 4;
    const int staged = rows_spanned(r0, r1, n_rows, RBLK);     // (all but the last of which end here)
    int row_pos[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
        const int i = u * NACHO_WAVE + lane;
        row_pos[u] = pos[r0 + (i < staged ? i : staged)];
    }
    const int pr0 = pos[r0], pr1 = pos[r1];
    // (kTable) this wavefront's share of the zeros, the first 64 rows of it
    const int share = kTable ? (n_rows + (int)gridDim.x - 1) / (int)gridDim.x : 0;
    const int zero0 = (int)blockIdx.x * share + lane, zero1 = min(((int)blockIdx.x + 1) * share, n_rows);
    int za = 0, zb = 1;
    if (kTable) {
        za = pos[zero0 < n_rows ? zero0 : n_rows];
        zb = pos[zero0 + 1 < n_rows ? zero0 + 1 : n_rows];
    }
    if (!kTable && last >= 0) {
#pragma unroll
        for (int j = 0; j < kIter; ++j) xv[j] = x[c[j]];
    }
    const bool has_head = n0 > pr0;                    // row r0 started in an earlier partition
    const int next_first = (n1 > pr1) ? r1 + 1 : r1;   // first row that starts after this partition
    const int nrows = next_first - r0;                 // rows overlapping or starting here
    int nr = nrows < RBLK ? nrows : RBLK;
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
        static_assert(kAhead * NACHO_WAVE <= RBLK, "every lane has a word to write");
        spos[u * NACHO_WAVE + lane] = row_pos[u];      // (what lies past the last row nobody reads)
    }
    for (int i0 = kAhead * NACHO_WAVE; i0 <= staged; i0 += kAhead * NACHO_WAVE) {
        int more[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int i = i0 + u * NACHO_WAVE + lane;
            more[u] = pos[r0 + (i < staged ? i : staged)];
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int i = i0 + u * NACHO_WAVE + lane;
            spos[i < staged ? i : staged] = more[u];
        }
    }
    if (kTable || last >= 0) {
#pragma unroll
        for (int j = 0; j < kIter; ++j) prod[j * NACHO_WAVE + lane] = v[j] * xv[j];
    }
    wave_sync();
    if (kTable) {
        if (zero0 < zero1 && za == zb) y[zero0] = T(0);
        if (share > NACHO_WAVE) {                      // (uniform)
            int a[kZeroRows / NACHO_WAVE - 1], b[kZeroRows / NACHO_WAVE - 1];
#pragma unroll
            for (int u = 0; u < kZeroRows / NACHO_WAVE - 1; ++u) {
                const int z = zero0 + (u + 1) * NACHO_WAVE;
                a[u] = pos[z < n_rows ? z : n_rows];
                b[u] = pos[z + 1 < n_rows ? z + 1 : n_rows];
            }
#pragma unroll
            for (int u = 0; u < kZeroRows / NACHO_WAVE - 1; ++u) {
                const int z = zero0 + (u + 1) * NACHO_WAVE;
                if (z < zero1 && a[u] == b[u]) y[z] = T(0);
            }
        }
        if (lane == 0) {
            // the partition table: this boundary, and the end
            coord[2 * p] = r0;
            coord[2 * p + 1] = r0 < n_rows && p > 0 ? c[0] : 0;
            posn[2 * p] = r0;
            posn[2 * p + 1] = p == 0 ? 0 : (r0 < n_rows ? n0 : nnz);
            cost[p] = n0;
            if (p == (int)gridDim.x - 1) {
                coord[2 * p + 2] = n_rows;
                coord[2 * p + 3] = 0;
                posn[2 * p + 2] = n_rows;
                posn[2 * p + 3] = nnz;
                cost[p + 1] = nnz;
            }
        }
    }

    // (unsigned: the block behind the last one may start past 2^31)
    for (unsigned rb = 0; rb < (unsigned)nrows; rb += RBLK) {
        if (rb > 0) {
            nr = nrows - (int)rb < RBLK ? nrows - (int)rb : RBLK;
            wave_sync();
            for (int i = lane; i <= nr; i += NACHO_WAVE) spos[i] = pos[r0 + (int)rb + i];
            wave_sync();
            // A block of rows without entries: their zeros are written elsewhere (by the partition
            // kernel, or above), so the wavefront steps over them, however many there are.
            const int q = spos[0];
            if (q == spos[nr]) {
                if (q >= n1) break;                     // every product of the partition is summed
                rb = (unsigned)(first_row_past(pos, r0 + (int)rb + nr, r0 + nrows, q) - r0) - RBLK;
                continue;
            }
        }
        for (int rr0 = 0; rr0 < nr; rr0 += NACHO_WAVE) {
            const int rr = rr0 + lane;
            const bool valid = rr < nr;
            const int a = valid ? spos[rr] : 0;
            const int b = valid ? spos[rr + 1] : 0;
            const int lo = (a > n0 ? a : n0) - a0;
            const int hi = (b < n1 ? b : n1) - a0;
            const int len = valid && hi > lo ? hi - lo : 0;
            T sum = T(0);
            if (len < kLongRow)
                for (int i = lo; i < lo + len; i += 4) {
                    T t[4];                            // (the words past the row are there: the slack of prod)
#pragma unroll
                    for (int u = 0; u < 4; ++u) t[u] = prod[i + u];
#pragma unroll
                    for (int u = 0; u < 4; ++u) sum += i + u < lo + len ? t[u] : T(0);
                }
            unsigned long long heavy = __ballot(len >= kLongRow);
            while (heavy) {
                const int L = __ffsll((long long)heavy) - 1;
                heavy &= heavy - 1;
                const int llo = __builtin_amdgcn_readlane(lo, L), lhi = __builtin_amdgcn_readlane(hi, L);
                T s = T(0);
#pragma unroll 4
                for (int i = llo + lane; i < lhi; i += NACHO_WAVE) s += prod[i];
                s = dpp_wave_sum(s);                   // (in lane 63)
                s = last_lane(s);
                if (lane == L) sum = s;
            }
            if (valid) {
                const int r = r0 + (int)rb + rr;
                if (has_head && r == r0) carry_val[p] = sum;
                else y[r] = sum;
            }
        }
    }
    if (lane == 0) carry_row[p] = has_head ? r0 : -1;
    wave_end(wlog, blockIdx.x, stamp, (uint32_t)(n1 - n0), (uint32_t)nrows);
}

// Carry fix-up, one lane per partition.  The carries of a row sit in
// consecutive partitions; the wavefront that holds the first carry of a row adds
// the whole run to y[row]: a segmented sum over its own 64 lanes, plus a walk
// over the following partitions when the run goes on past the wavefront's last
// lane.  One writer per row and a fixed order of additions.
template <typename T>
__global__ void __launch_bounds__(256)
spmv_fixup_kernel(T *__restrict__ y, int P, const T *__restrict__ carry_val,
                  const int32_t *__restrict__ carry_row, const int32_t *__restrict__ pos, int grain)
{
    const int p = (int)((int64_t)blockIdx.x * blockDim.x + threadIdx.x);
    const int lane = lane_id();
    const int p_first = p - lane;                      // partition of lane 0
    if (p_first >= P) return;                          // whole wavefront leaves together
    // (all three asked for at once: a partition without a carry has some words there)
    const int at = p < P ? p : P - 1;
    int r = carry_row[at];
    T v = carry_val[at];
    const int row_before = carry_row[p_first > 0 ? p_first - 1 : 0];
    if (p >= P) r = -1;
    if (r < 0) v = T(0);
    int before = __builtin_amdgcn_update_dpp(0, r, 0x138, 0xf, 0xf, false);    // wave_shr:1
    if (lane == 0) before = p_first > 0 ? row_before : -1;
    const bool head = r >= 0 && r != before;           // first carry of its row
    const bool first_here = r != before || lane == 0;  // first lane of its segment in this wavefront
    const unsigned long long starts = __ballot(first_here);
    const unsigned long long upto = low_bits(lane + 1);
    const int start = 63 - __clzll((long long)(starts & upto));
    const unsigned long long after = starts & ~upto;
    const int end = after ? __ffsll((long long)after) - 2 : NACHO_WAVE - 1;   // last lane of the segment
    // inclusive sum inside the segment, by DPP moves (a shuffle goes through the LDS unit, and nothing hides the chain of
    // them here; with the longer batches below 40,000 non-zeros: 10.4 to 9.9 us, 5M: 31.3 to 30.3, 50M: 308 to 302)
    auto add = [&](T left, bool same) { v += same ? left : T(0); };
    add(dpp_moved<0x111, 0xf>(v), lane - 1 >= start);                      // row_shr:1, 2, 4, 8: inside 16 lanes
    add(dpp_moved<0x112, 0xf>(v), lane - 2 >= start);
    add(dpp_moved<0x114, 0xf>(v), lane - 4 >= start);
    add(dpp_moved<0x118, 0xf>(v), lane - 8 >= start);
    add(dpp_moved<0x142, 0xa>(v), start < (lane & ~15));                   // row_bcast:15 into rows 1 and 3
    add(dpp_moved<0x143, 0xc>(v), start < NACHO_WAVE / 2);                 // row_bcast:31 into rows 2 and 3
    const unsigned long long heads = __ballot(head);
    auto owned_from = [&](int first) { return bit_at(heads, first); };     // the run from that lane on starts in this wavefront
    const bool owned = owned_from(start);
    // a run that reaches the last lane may go on in the next wavefronts
    const int r_last = __builtin_amdgcn_readlane(r, NACHO_WAVE - 1);
    const bool last_owned = owned_from(__builtin_amdgcn_readlane(start, NACHO_WAVE - 1));
    // (the writer's element of y is requested now, beside the loads of the tail)
    const bool writer = r >= 0 && owned && lane == end;
    const T y_old = writer ? y[r] : T(0);
    T tail = T(0);
    if (r_last >= 0 && last_owned && grain > 0) {
        // fixed-grain partitions: the carries of row r come from the partitions that
        // start strictly inside it, floor(pos[r] / grain) + 1 .. ceil(pos[r+1] / grain) - 1,
        // so the rest of the run is known without looking: independent loads, eight or
        // (long runs: a row of a million non-zeros has 2000 carries) 32 chunks of 64 in
        // flight, added in a fixed order
        int last = shares_before(pos[r_last + 1], grain) - 1;          // (pos[0] = 0)
        if (last > P - 1) last = P - 1;
        T acc[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc[u] = T(0);
        int q0 = p_first + NACHO_WAVE;
        auto chunks = [&](auto batch_tag) {
            constexpr int kBatch = decltype(batch_tag)::value;
            T t[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int q = q0 + u * NACHO_WAVE + lane;
                t[u] = q <= last ? carry_val[q] : T(0);
            }
#pragma unroll
            for (int u = 0; u < kBatch; ++u) acc[u & 7] += t[u];
            q0 += kBatch * NACHO_WAVE;
        };
        while (last - q0 >= 8 * NACHO_WAVE) chunks(std::integral_constant<int, 32>());
        if (q0 <= last) chunks(std::integral_constant<int, 8>());
        tail = last_lane(dpp_wave_sum(((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]))));
    } else if (r_last >= 0 && last_owned) {
        // chunks of 64 partitions, loaded in batches: two chunks first (most runs end
        // there), then sixteen at a time (a row of a million non-zeros has thousands of
        // carries; every batch is one round trip)
        int e = p_first + NACHO_WAVE;
        bool more = true;
        auto walk = [&](auto batch_tag) {
            constexpr int kBatch = decltype(batch_tag)::value;
            int rr[kBatch];
            T vv[kBatch];
#pragma unroll
            for (int c = 0; c < kBatch; ++c) {
                const int q = e + c * NACHO_WAVE + lane;
                rr[c] = q < P ? carry_row[q] : -1;
                vv[c] = q < P ? carry_val[q] : T(0);
            }
#pragma unroll
            for (int c = 0; c < kBatch; ++c) {
                if (!more) break;
                const unsigned long long m = __ballot(rr[c] == r_last);
                const int cnt = m == ~0ull ? NACHO_WAVE : __ffsll((long long)~m) - 1;   // leading lanes of the run
                tail += wave_sum(lane < cnt ? vv[c] : T(0));
                more = cnt == NACHO_WAVE;
            }
            e += kBatch * NACHO_WAVE;
        };
        walk(std::integral_constant<int, 2>());
        while (more) walk(std::integral_constant<int, 16>());
    }
    if (writer) y[r] = y_old + (v + (end == NACHO_WAVE - 1 ? tail : T(0)));
}

// Non-zeros of a partition (and row positions staged at a time), at most.
constexpr int kGrainF64 = 512, kGrainF32 = 1024, kShortGrainF32 = 512;

}  // namespace

int spmv_capacity(int dtype) { return dtype == NACHO_F64 ? kGrainF64 : kGrainF32; }

// Floats, P = 0.  A wavefront's loads, sums and stores are one chain of latencies, so twice as many wavefronts, half as long, are faster
// where few are in flight and where the chain has many rows to sum (partitions of 1024 and of 512 non-zeros, us: 50,000, 5 a row 11.2
// and 8.8; 2M, 5, 10, 20 a row 25.7, 21.0, 16.4 and 22.1, 18.6, 15.7; 10M, 5, 10, 20, 40 a row 78.6, 59.2, 49.5, 45.6 and 72.5, 54.9,
// 46.2, 43.0).  Rows of many non-zeros are summed at a stretch, and 5000 wavefronts of 1024 non-zeros hold more loads in flight than 8192
// of 512: 60, 100, 300 a row, 4M 20.9, 19.6, 18.0 and 22.6, 21.7, 19.8, 5M 24.6, 23.5, 21.3 and 26.8, 25.4, 23.0; 1.5M 12.2, 11.4, 10.5
// and 11.9, 11.3, 10.6.  Past one round of wavefronts of either length that is over, and long ones, which such calls still take, lose
// 3 to 4 % where rows are not very long: 8M 36.2, 34.6, 31.2 and 35.1, 34.4, 32.7, 50M 178, 170, 162 and 173, 163, 157.
// Tables of a caller's P and of the row-aware cost have up to 1024.
int64_t spmv_grain(int dtype, int64_t nnz, int64_t n_rows)
{
    if (dtype == NACHO_F64) return kGrainF64;
    return nnz >= 1'400'000 && nnz >= 48 * n_rows ? kGrainF32 : kShortGrainF32;
}

// Small calls do without a partition kernel: its place in the stream (a launch and 3 us) is a third of what such a call takes, and the
// wavefronts' search for their rows travels beside their non-zeros.  Short partitions of floats count half, whose search is a larger
// share of a wavefront.  Up to 1024 partitions, counted so, with any x; past them partitions inside long rows would have to be dealt out
// by XCD, which this form does not do, unless x fits an L2 of 4 MiB (50M non-zeros: 298 to 467 us without).  With and without the partition
// kernel, us:
//   Up to 4096 partitions, whatever their length, x of 4 MiB: doubles, x of 2.4 to 3.2 MB, 1.5M 22.7 and 21.2, 2M 26.6 and 25.5.
//   Past 4096 doubles with x of 2.5 MiB, which leaves L2 for the rest, up to 10240 partitions: x of 0.7 and 2 MB, 5M (9766) 34.0, 37.5 and
//   32.1, 37.5; 8M (15625) 47.9 and 49.3; x of 2.4 to 3.2 MB, 3M (5860) 30.0 and 28.7, 4M (7813) 35.9 and 36.5; of 4.8 MB, 3M 33.1 and 34.4.
//   Past 4096 floats with x of 4 MiB and 131,072 rows up to 10240 short or 8192 long ones: level while rows are few (short ones, 20 a row,
//   2.6M 20.6 and 20.0, 3M 21.7 and 21.8, 6M 31.9 and 31.3), and the search loses where they are not (10 a row, 3M 23.6 and 24.1, 5M 31.7
//   and 34.1).
// With more than 256 rows a partition (counted as above), which the wavefronts could not look after in one batch of loads each, the
// partition kernel writes the zeros, a row a thread (40,000 non-zeros in the first 4096 of 131072 rows: 63 to 17 us).
bool spmv_whole(int dtype, int64_t nnz, int64_t grain, int64_t P, int64_t n_rows, int64_t x_bytes)
{
    if (nnz == 0) return false;                        // (its wavefronts expect non-zeros)
    const bool halves = dtype == NACHO_F32 && grain < kGrainF32;
    const int64_t parts = halves ? (P + 1) / 2 : P;
    if (n_rows > parts * kZeroRows) return false;
    if (parts <= 1024) return true;
    if (P <= 4096) return x_bytes <= (4 << 20);
    if (dtype == NACHO_F64) return P <= 10240 && x_bytes <= (5 << 19);
    return n_rows <= (1 << 17) && parts <= (halves ? 5120 : 8192) && x_bytes <= (4 << 20);
}

hipError_t launch_spmv_exec(int dtype, const int32_t *pos, const int32_t *crd, const void *val,
                            const void *x, void *y, int64_t n_rows, int64_t nnz,
                            int32_t *coord, int32_t *posn, int64_t *cost, int64_t P,
                            void *carry_val, int32_t *carry_row, int64_t grain, SpmvForm form, hipStream_t stream)
{
#define NACHO_SPMV_LAUNCH(T, G, R, DEALT, FUSED, TABLE)                                                        \
    hipLaunchKernelGGL((spmv_exec_kernel<T, G, R, DEALT, FUSED, TABLE>), dim3((unsigned)P), dim3(NACHO_WAVE), 0, stream, \
                       pos, crd, (const T *)val, (const T *)x, (T *)y, (int)nnz, coord, posn, cost, (T *)carry_val,    \
                       carry_row, (int)n_rows, (int)grain, nacho_host::wave_log())
#define NACHO_SPMV_GRAIN(T, G)                                                                  \
    case SPMV_DEALT: NACHO_SPMV_LAUNCH(T, G, G, true, false, false); break;                     \
    case SPMV_SEARCH: NACHO_SPMV_LAUNCH(T, G, G, true, true, false); break;                     \
    case SPMV_WHOLE: NACHO_SPMV_LAUNCH(T, G, G, false, true, true); break;
#define NACHO_SPMV_FORM(T, G)                                                                   \
    switch (form) {                                                                             \
    case SPMV_TABLE: NACHO_SPMV_LAUNCH(T, G, G, false, false, false); break;                    \
    NACHO_SPMV_GRAIN(T, G)                                                                      \
    }
    if (dtype == NACHO_F64) { NACHO_SPMV_FORM(double, kGrainF64) }
    else if (grain == kShortGrainF32) {
        switch (form) {
        case SPMV_TABLE: return hipErrorInvalidValue;      // (has no grain)
        NACHO_SPMV_GRAIN(float, kShortGrainF32)
        }
    } else { NACHO_SPMV_FORM(float, kGrainF32) }
#undef NACHO_SPMV_GRAIN
#undef NACHO_SPMV_FORM
#undef NACHO_SPMV_LAUNCH
    return hipGetLastError();
}

namespace {
__global__ void __launch_bounds__(256) zero_words_kernel(uint32_t *__restrict__ dst, int64_t n_words)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_words; i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = 0u;
}
}  // namespace

// y = 0 (the fused form has no partition kernel to write the zeros of the rows A stores nothing in)
hipError_t launch_zero_vector(int dtype, void *y, int64_t n, hipStream_t stream)
{
    const int64_t words = n * (dtype == NACHO_F64 ? 2 : 1);
    if (words == 0) return hipSuccess;
    int64_t blocks = (words + 255) / 256;
    if (blocks > 256 * 64) blocks = 256 * 64;
    hipLaunchKernelGGL(zero_words_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, (uint32_t *)y, words);
    return hipGetLastError();
}

hipError_t launch_spmv_fixup(int dtype, void *y, int64_t P, const void *carry_val,
                             const int32_t *carry_row, const int32_t *pos, int64_t grain, hipStream_t stream)
{
    const unsigned grid = (unsigned)((P + 255) / 256);
    if (dtype == NACHO_F64)
        hipLaunchKernelGGL((spmv_fixup_kernel<double>), dim3(grid), dim3(256), 0, stream,
                           (double *)y, (int)P, (const double *)carry_val, carry_row, pos, (int)grain);
    else
        hipLaunchKernelGGL((spmv_fixup_kernel<float>), dim3(grid), dim3(256), 0, stream,
                           (float *)y, (int)P, (const float *)carry_val, carry_row, pos, (int)grain);
    return hipGetLastError();
}

}  // namespace nacho
