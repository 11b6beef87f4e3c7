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
    // Which partition this workgroup executes: those inside one long row are dealt out by XCD, so that the gathers of an XCD
    // stay inside one eighth of x, which its L2 holds (all of x it does not).
    int p = blockIdx.x;
    // (fused search) the rows and positions of the boundaries p and p + 1
    int r0 = 0, r1 = 0, n0 = 0, n1 = 0;
    auto boundaries = [&]() {
        const int base = pos[0];
        const long long Qa = (long long)p * grain, Qb = Qa + grain;
        n0 = base + (int)(Qa < nnz ? Qa : nnz);
        n1 = base + (int)(Qb < nnz ? Qb : nnz);
        rows_holding(pos, n_rows, n0, n1, r0, r1);
        if (p == 0) r0 = 0;
        else if (Qa >= nnz) r0 = n_rows;
        if (Qb >= nnz) r1 = n_rows;
    };
    if (kFused) boundaries();
    if (kDealt) {
        const int r = kFused ? r0 : coord[2 * p];
        if (r < n_rows) {
            const int base = pos[0];
            p = dealt_partition(p, pos[r] - base, pos[r + 1] - base, grain);
        }
    }
    // k = 1, d = 2: coord[b*2 + 0] = row, posn[b*2 + 1] = position in crd/val
    if (kFused) {
        if (p != (int)blockIdx.x) boundaries();
        if (kTable && lane == 0) {
            // the partition table: this boundary, and the end
            coord[2 * p] = r0;
            coord[2 * p + 1] = r0 < n_rows ? (p == 0 ? 0 : crd[n0]) : 0;
            posn[2 * p] = r0;
            posn[2 * p + 1] = p == 0 ? 0 : (r0 < n_rows ? n0 : nnz);
            cost[p] = n0 - pos[0];
            if (p == (int)gridDim.x - 1) {
                coord[2 * p + 2] = n_rows;
                coord[2 * p + 3] = 0;
                posn[2 * p + 2] = n_rows;
                posn[2 * p + 3] = nnz;
                cost[p + 1] = nnz;
            }
        }
    } else {
        r0 = coord[2 * p]; r1 = coord[2 * p + 2];
        n0 = posn[2 * p + 1]; n1 = posn[2 * p + 3];
    }
    const int pr0 = pos[r0], pr1 = pos[r1];
    const bool has_head = n0 > pr0;                    // row r0 started in an earlier partition
    const int next_first = (n1 > pr1) ? r1 + 1 : r1;   // first row that starts after this partition
    const int nrows = next_first - r0;                 // rows overlapping or starting here
    const int a0 = n0;                                 // prod[i] belongs to position a0 + i
    // pos entries of the first row block, requested before the streamed data
    int nr = nrows < RBLK ? nrows : RBLK;
    if (nrows > 0)
        for (int i = lane; i <= nr; i += NACHO_WAVE) spos[i] = pos[r0 + i];

    // Lane l takes positions n0 + l, n0 + 64 + l, ...: consecutive lanes hold
    // consecutive non-zeros, so inside a dense row the 64 gathers of one
    // instruction fall into few cache lines of x (columns are sorted).  All
    // streamed loads are issued before the first gather, all gathers before the
    // first LDS store, so one wavefront keeps its whole window in flight.
    // (places are compared, not positions: the last ones may lie past 2^31)
    constexpr int kIter = G / NACHO_WAVE;
    const int left = n1 - n0 - lane;
    int c[kIter];
    T v[kIter];
#pragma unroll
    for (int j = 0; j < kIter; ++j) {
        c[j] = 0;
        v[j] = T(0);
        if (j * NACHO_WAVE < left) {
            const int idx = n0 + j * NACHO_WAVE + lane;
            c[j] = __builtin_nontemporal_load(crd + idx);
            v[j] = __builtin_nontemporal_load(val + idx);
        }
    }
    T xv[kIter];
#pragma unroll
    for (int j = 0; j < kIter; ++j) xv[j] = j * NACHO_WAVE < left ? x[c[j]] : T(0);
    if (kTable) {
        const int share = (n_rows + (int)gridDim.x - 1) / (int)gridDim.x;
        const int z = (int)blockIdx.x * share + lane, z_end = min((int)(blockIdx.x + 1) * share, n_rows);
        int a[kZeroRows / NACHO_WAVE], b[kZeroRows / NACHO_WAVE];
#pragma unroll
        for (int u = 0; u < kZeroRows / NACHO_WAVE; ++u) {
            a[u] = 0;
            b[u] = 1;
            if (z + u * NACHO_WAVE < z_end) { a[u] = pos[z + u * NACHO_WAVE]; b[u] = pos[z + u * NACHO_WAVE + 1]; }
        }
#pragma unroll
        for (int u = 0; u < kZeroRows / NACHO_WAVE; ++u)
            if (a[u] == b[u]) y[z + u * NACHO_WAVE] = T(0);
    }
#pragma unroll
    for (int j = 0; j < kIter; ++j)
        if (j * NACHO_WAVE < left) prod[j * NACHO_WAVE + lane] = v[j] * xv[j];
    __syncthreads();

    for (int rb = 0; rb < nrows; rb += RBLK) {
        if (rb > 0) {
            nr = nrows - rb < RBLK ? nrows - rb : RBLK;
            __syncthreads();
            for (int i = lane; i <= nr; i += NACHO_WAVE) spos[i] = pos[r0 + rb + i];
            __syncthreads();
            // A block of rows without entries: their zeros are written elsewhere (by the partition
            // kernel, or above), so the wavefront steps over them, however many there are.
            const int q = spos[0];
            if (q == spos[nr]) {
                if (q >= n1) break;                     // every product of the partition is summed
                rb = first_row_past(pos, r0 + rb + nr, r0 + nrows, q) - r0 - RBLK;
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
                const int r = r0 + rb + rr;
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
    const int r = p < P ? carry_row[p] : -1;
    T v = r >= 0 ? carry_val[p] : T(0);
    int before = __builtin_amdgcn_update_dpp(0, r, 0x138, 0xf, 0xf, false);    // wave_shr:1
    if (lane == 0) before = p_first > 0 ? carry_row[p_first - 1] : -1;
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
        const int base = pos[0];
        int last = shares_before(pos[r_last + 1] - base, grain) - 1;
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
// where few are in flight and where the chain has many rows to sum (partitions of 1024 and of 512 non-zeros, us: 0.1M, 6, 60, 300
// a row 13.0, 9.3, 9.2 and 9.9, 8.1, 8.0; 2M, 6, 10, 20 a row 24.9, 23.5, 18.8 and 22.5, 21.3, 17.4; 10M 71.7, 62.7, 54.8 and 68.4, 60.3, 52.9).
// Rows of many non-zeros are summed at a stretch, and a large call is as long as its loads, of which 5000 wavefronts of 1024 non-zeros
// hold more in flight than 8192 of 512: 60, 100, 300 a row, 4M 24.6, 23.0, 19.7 and 25.8, 24.5, 21.3, 6M 32.8, 31.3, 27.2 and 34.8, 34.2, 30.8, 50M
// 196, 189, 180 and 200, 193, 184; but 1M 11.3, 10.9, 10.5 and 10.4, 10.1, 9.7.  The lines lie between: 40 a row 0.97 to 1.03 of the time with 512 (slower at
// 4M and 5M), 1.5M with 60, 100, 300 a row 1.00, 1.05, 0.96.  Tables of a caller's P and of the row-aware cost have up to 1024 (two non-zeros a row as cost, 5M, 10 a row 39.9 and 46.2).
int64_t spmv_grain(int dtype, int64_t nnz, int64_t n_rows)
{
    if (dtype == NACHO_F64) return kGrainF64;
    return nnz >= 1'400'000 && nnz >= 48 * n_rows ? kGrainF32 : kShortGrainF32;
}

// Small calls do without a partition kernel.  Its place in the stream (a launch and 3 us) is a third of what such a
// call takes, while the wavefronts find their rows in two or three rounds of loads that hit the cache (40,000
// non-zeros: 9.3 us in all; 1M: 16.8 to 15.4; 5M: 33.2 to 32.4).  Past a thousand partitions only while x fits an L2:
// partitions inside long rows are not dealt out by XCD in this form (50M non-zeros: 309 to 469 us without).  With more
// rows than the wavefronts can look after in one batch of loads each the partition kernel writes the zeros, a row a
// thread (40,000 non-zeros in the first 4096 of 131072 rows: 63 to 17 us).  The lines are in partitions of fp64 and of long ones of fp32; short
// ones count half, whose search takes a larger share of a wavefront (with and without the partition kernel 31.6 and 31.0 us for 5M
// non-zeros, 34.8 and 34.8 for 6M, 42.2 and 43.5 for 8M).
bool spmv_whole(int dtype, int64_t grain, int64_t P, int64_t n_rows, int64_t x_bytes)
{
    const bool halves = dtype == NACHO_F32 && grain < kGrainF32;
    const int64_t parts = halves ? (P + 1) / 2 : P;
    return n_rows <= (1 << 17) && n_rows <= parts * kZeroRows && (parts <= 1024 || (parts <= (halves ? 5120 : 8192) && x_bytes <= (4 << 20)));
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
