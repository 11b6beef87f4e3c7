// SpMM execution, C = A B with A in CSR and B, C dense row-major: loop order i -> j -> k with the dense k
// innermost (the broadcast rule of Section 4.2.2 scales the cost of every stored non-zero by n, so the
// partitions are those of SpMV), one wavefront per partition.
//
// What bounds it: large matrices the rows of B (30M non-zeros x 256 bytes: 6.6 TB/s out of the last-level cache and
// memory), all others how many of those rows are on their way at a time.  So a row of B is not spread over the whole
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

// V elements of a row of B or C; in memory they are aligned as one element is (16-byte loads and stores need no more).
template <typename T, int V> struct Piece {
    typedef T type __attribute__((ext_vector_type(V)));
    typedef type mem __attribute__((aligned(sizeof(T))));
};

// W lanes a row, CPL pieces of V elements a lane.  kWhole: there is no partition kernel; the wavefront searches its
// rows, stores its part of the partition table and writes the zeros of its empty rows.
template <typename T, int V, int W, int CPL, bool kWhole>
__global__ void __launch_bounds__(NACHO_WAVE)
spmm_exec_kernel(const int32_t *__restrict__ pos, const int32_t *__restrict__ crd, const T *__restrict__ val,
                 const T *__restrict__ B, int n, int span, int64_t ldb, T *__restrict__ C, int64_t ldc,
                 int32_t *__restrict__ coord, int32_t *__restrict__ posn, int64_t *__restrict__ cost,
                 T *__restrict__ carry_val, int32_t *__restrict__ carry_row, int n_rows, int nnz, int grain,
                 int64_t cost_scale, WaveLog wlog)
{
    typedef typename Piece<T, V>::type P;
    typedef typename Piece<T, V>::mem PM;
    constexpr int NG = NACHO_WAVE / W;         // groups
    constexpr int kSlots = kGrain + 4 * NG;    // a group's stretch is followed by 4 words (banks of their own for every group)
    constexpr int kIter = kGrain / NACHO_WAVE;
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

    const int p = blockIdx.x, lane = threadIdx.x, g = lane / W, gl = lane & (W - 1);
    int r0, r1, n0, n1;
    if (kWhole) {
        const int base = pos[0];
        const long long Qa = (long long)p * grain, Qb = Qa + grain;
        n0 = base + (int)(Qa < nnz ? Qa : nnz);
        n1 = base + (int)(Qb < nnz ? Qb : nnz);
        rows_holding(pos, n_rows, n0, n1, r0, r1);
        if (p == 0) r0 = 0;
        else if (Qa >= nnz) r0 = n_rows;
        if (Qb >= nnz) r1 = n_rows;
    } else {
        r0 = coord[2 * p]; r1 = coord[2 * p + 2];
        n0 = posn[2 * p + 1]; n1 = posn[2 * p + 3];
    }
    const int len = n1 - n0;
    const int S = ((len + NG - 1) / NG + 3) & ~3;      // a group's stretch
    const int left = len - g * S, items = left < 0 ? 0 : (left < S ? left : S);
    const int base = g * (S + 4);                      // its first slot
    // everything is asked for before the first wait: the stretch, the ends of the rows
    int32_t c_in[kIter];
    T v_in[kIter];
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
    const int pr0 = pos[r0], pr1 = pos[r1];
    const bool has_head = n0 > pr0;                    // row r0 started in an earlier partition
    const int next_first = n1 > pr1 ? r1 + 1 : r1;     // first row that starts after this partition
    int row = r0 + lane, row_a = 0, row_b = 0;
    if (row < next_first) { row_a = pos[row]; row_b = pos[row + 1]; }
    if (kWhole && lane == 0 && blockIdx.y == 0) {
        coord[2 * p] = r0;
        coord[2 * p + 1] = r0 < n_rows ? (p == 0 ? 0 : crd[n0]) : 0;
        posn[2 * p] = r0;
        posn[2 * p + 1] = p == 0 ? 0 : (r0 < n_rows ? n0 : nnz);
        cost[p] = (int64_t)(n0 - pos[0]) * cost_scale;
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
            s_val[base + i] = v_in[j];
            s_row[base + i] = -1;
        }
    }
    __syncthreads();
    if (kWhole) {
        // zeros of empty rows: every wavefront looks after an equal share of all rows, 64 of them at a time
        const int z0 = (int)((int64_t)n_rows * p / gridDim.x), z1 = (int)((int64_t)n_rows * (p + 1) / gridDim.x);
        for (int z = z0; z < z1; z += NACHO_WAVE) {
            const bool is_empty = z + lane < z1 && pos[z + lane] == pos[z + lane + 1];
            const unsigned long long empty = __ballot(is_empty);
            if (empty == 0ull) continue;
            for (int i = g; i < NACHO_WAVE; i += NG)
                if (bit_at(empty, i)) {
#pragma unroll
                    for (int c = 0; c < CPL; ++c)
                        if (mine[c]) *reinterpret_cast<PM *>(C + (int64_t)(z + i) * ldc + col[c]) = P(T(0));
                }
        }
    }
    const float per_S = 1.0f / (float)S;
    for (;;) {                                         // rows, 64 at a time
        const bool is_row = row < next_first;
        if (is_row && row_b > row_a && row_a >= n0) {
            const int i = row_a - n0;                  // (< len: the row starts in this partition)
            const int at = (int)(((float)i + 0.5f) * per_S);       // i / S
            s_row[i + 4 * at] = row;
        }
        const int next = __builtin_amdgcn_readfirstlane(row) + NACHO_WAVE;
        if (next >= next_first) break;
        int from = next;
        if (__ballot(row_b > row_a) == 0ull) {
            // 64 rows without an entry: however many there are, stepped over
            const int q = __builtin_amdgcn_readfirstlane(row_b);
            if (q >= n1) break;
            from = first_row_past(pos, next, next_first, q);
        }
        row = from + lane;
        row_a = row_b = 0;
        if (row < next_first) { row_a = pos[row]; row_b = pos[row + 1]; }
    }
    __syncthreads();

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
    __syncthreads();
    P *s_head = reinterpret_cast<P *>(smem);
#pragma unroll
    for (int c = 0; c < CPL; ++c) s_head[c * NACHO_WAVE + lane] = head[c];
    __syncthreads();
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
    if (blockIdx.y == 0) wave_end(wlog, p, stamp, (uint32_t)len, (uint32_t)(next_first - r0));
}

// Carry fix-up: 16 lanes and up to 64 columns per partition, 16 partitions per workgroup.  The carries of a row lie in
// consecutive partitions; the lanes of the first one add the run to the row of C.  A run of more than kShort carries
// (there is at most one per workgroup: it is longer than the workgroup's partitions) is added by the whole workgroup,
// every group a sixteenth of it: the largest row of 30M non-zeros has 488, which one wavefront, a row of carries at a
// time, took 35 us for.  The order of the additions is fixed.
constexpr int kFixLanes = 16, kFixCols = 4, kFixGroups = 256 / kFixLanes, kShort = 32;

template <typename T>
__global__ void __launch_bounds__(256)
spmm_fixup_kernel(T *__restrict__ C, int64_t ldc, int n, int P, const T *__restrict__ carry_val,
                  const int32_t *__restrict__ carry_row, const int32_t *__restrict__ pos,
                  const int32_t *__restrict__ posn, int grain)
{
    static_assert(kShort >= kFixGroups, "one long run per workgroup");
    __shared__ T part[kFixGroups][kFixLanes * kFixCols];
    __shared__ int s_first, s_end, s_row;
    const int g = threadIdx.x / kFixLanes, gl = threadIdx.x & (kFixLanes - 1);
    const int p = blockIdx.x * kFixGroups + g;
    const int j0 = blockIdx.y * (kFixLanes * kFixCols) + gl;
    if (threadIdx.x == 0) s_first = -1;
    __syncthreads();
    const int r = p < P ? carry_row[p] : -1;
    const bool first = r >= 0 && (p == 0 || carry_row[p - 1] != r);
    int e = p + 1;
    if (first) {
        // the run ends with the last partition that starts inside the row
        const int row_end = pos[r + 1];
        if (grain > 0) e = shares_before(row_end - pos[0], grain);
        else {
            int lo = p + 1, hi = P;                    // the first partition that starts at or behind the row's end
            while (lo < hi) {
                const int mid = lo + ((hi - lo) >> 1);
                if (posn[2 * mid + 1] < row_end) lo = mid + 1; else hi = mid;
            }
            e = lo;
        }
        e = e < P ? e : P;
    }
    // carries q, q + step, ... below `to`, eight of them in flight
    auto sum = [&](int q, int to, int step, T (&x)[kFixCols]) {
#pragma unroll
        for (int c = 0; c < kFixCols; ++c) x[c] = T(0);
        for (; q < to; q += 8 * step) {
            T t[8][kFixCols];
#pragma unroll
            for (int u = 0; u < 8; ++u)
#pragma unroll
                for (int c = 0; c < kFixCols; ++c) {
                    t[u][c] = T(0);
                    if (q + u * step < to && j0 + c * kFixLanes < n)
                        t[u][c] = carry_val[(int64_t)(q + u * step) * n + j0 + c * kFixLanes];
                }
#pragma unroll
            for (int u = 0; u < 8; ++u)
#pragma unroll
                for (int c = 0; c < kFixCols; ++c) x[c] += t[u][c];
        }
    };
    T x[kFixCols];
    if (first && e - p <= kShort) {
        sum(p, e, 1, x);
#pragma unroll
        for (int c = 0; c < kFixCols; ++c)
            if (j0 + c * kFixLanes < n) C[(int64_t)r * ldc + j0 + c * kFixLanes] += x[c];
    } else if (first && gl == 0) {
        s_first = p;
        s_end = e;
        s_row = r;
    }
    __syncthreads();
    if (s_first < 0) return;                           // (the whole workgroup)
    sum(s_first + g, s_end, kFixGroups, x);
#pragma unroll
    for (int c = 0; c < kFixCols; ++c) part[g][c * kFixLanes + gl] = x[c];
    __syncthreads();
    if (g < kFixCols && j0 + g * kFixLanes < n) {
        T y = T(0);
#pragma unroll
        for (int u = 0; u < kFixGroups; ++u) y += part[u][g * kFixLanes + gl];
        C[(int64_t)s_row * ldc + j0 + g * kFixLanes] += y;
    }
}

}  // namespace

int spmm_capacity() { return kGrain; }

// Non-zeros per partition when the caller leaves the partitioning to the library: enough wavefronts for the chip.
int spmm_grain(int64_t nnz, int units)
{
    const int64_t per = nnz / ((int64_t)units * 16);
    return per >= kGrain ? kGrain : (per < 64 ? 64 : (int)((per + 63) / 64 * 64));
}

// Fixed-grain calls do without a partition kernel: the wavefronts of the executing kernel find their rows in two to
// four rounds of loads, which hide behind each other, and its place in the stream is saved (100k non-zeros, n = 16:
// 13.4 to 11.2 us; 1.3M, n = 37: 75 to 72; 30M, n = 64: 1136 to 1125).  The zeros of empty rows are spread over the
// wavefronts; where that would be thousands of rows each, the partition kernel writes them.
bool spmm_whole(int64_t P, int64_t n_rows) { return n_rows <= P * 1024; }

hipError_t launch_spmm_exec(int dtype, const int32_t *pos, const int32_t *crd, const void *val,
                            const void *B, int n, int64_t ldb, void *C, int64_t ldc, int64_t n_rows, int64_t nnz,
                            int32_t *coord, int32_t *posn, int64_t *cost, int64_t P, void *carry_val,
                            int32_t *carry_row, int64_t grain, int64_t cost_scale, bool whole,
                            hipStream_t stream)
{
    const int V = dtype == NACHO_F64 ? 2 : 4;
    // stretches of up to 64 pieces of V columns, of about equal width
    const int pieces = n < V ? n : (n + V - 1) / V, stretches = (pieces + NACHO_WAVE - 1) / NACHO_WAVE;
    const int per = (pieces + stretches - 1) / stretches;
    const int span = n < V ? n : per * V;
#define NACHO_SPMM_LAUNCH(T, VV, W, CPL, WHOLE)                                                                         \
    hipLaunchKernelGGL((spmm_exec_kernel<T, VV, W, CPL, WHOLE>), dim3((unsigned)P, (unsigned)stretches), dim3(NACHO_WAVE), 0,  \
                       stream, pos, crd, (const T *)val, (const T *)B, n, span, ldb, (T *)C, ldc, coord, posn, cost,    \
                       (T *)carry_val, carry_row, (int)n_rows, (int)nnz, (int)grain, cost_scale, \
                       nacho_host::wave_log())
#define NACHO_SPMM_SHAPE(T, VV, W, CPL)                                                                                 \
    do {                                                                                                                \
        if (whole) NACHO_SPMM_LAUNCH(T, VV, W, CPL, true);                                                              \
        else NACHO_SPMM_LAUNCH(T, VV, W, CPL, false);                                                                   \
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
                             hipStream_t stream)
{
    constexpr int cols = kFixLanes * kFixCols;
    const dim3 grid((unsigned)((P + kFixGroups - 1) / kFixGroups), (unsigned)((n + cols - 1) / cols));
    if (dtype == NACHO_F64)
        hipLaunchKernelGGL((spmm_fixup_kernel<double>), grid, dim3(256), 0, stream, (double *)C, ldc,
                           n, (int)P, (const double *)carry_val, carry_row, pos, posn, (int)grain);
    else
        hipLaunchKernelGGL((spmm_fixup_kernel<float>), grid, dim3(256), 0, stream, (float *)C, ldc,
                           n, (int)P, (const float *)carry_val, carry_row, pos, posn, (int)grain);
    return hipGetLastError();
}

}  // namespace nacho
