// Launchers of the HIP kernels (one translation unit per kernel family).
#pragma once
#include "common.hpp"

namespace nacho {

// Algorithm 1 for boundaries 0..P.  `queries` (device, may be NULL) overrides
// the built-in queries; otherwise Q_p = min(p*grain, total) when grain > 0 and
// floor(p*total/P) when grain == 0 (total = total_unscaled * cost_scale).
// `clear_words` (may be NULL): n_clear 64-bit words the kernel sets to zero on the side, and
// `clear_status` (may be NULL) a status word it sets to NACHO_OK: the state of the kernels that
// follow it in a fused call.
// `row_cost` (one CSR operand with built-in queries only): every row costs that many units on top of its
// stored non-zeros (in the units of a non-zero before cost_scale); total_unscaled stays the non-zero count.
// `zero_rows` (may be NULL; one CSR operand with built-in queries only, i.e. the fused SpMV and
// SpMM calls): the kernel also sets to zero the rows of a dense result whose operand row is empty.
struct ZeroRows {
    void *base;          // row r of the result: `width` elements of `elem` bytes from base + r * ld * elem
    int64_t ld;
    int32_t width, elem;
};
hipError_t launch_partition(const DevOperands &ops, int64_t cost_scale, int64_t P, int64_t grain,
                            const int64_t *queries, int64_t total_unscaled,
                            int32_t *coord, int32_t *posn, int64_t *cost, hipStream_t stream,
                            unsigned long long *clear_words = nullptr, int64_t n_clear = 0,
                            int32_t *clear_status = nullptr, const ZeroRows *zero_rows = nullptr,
                            int64_t row_cost = 0);

hipError_t launch_partition_csr64(const int64_t *pos, const int32_t *crd, int64_t n_rows, int64_t nnz, int64_t P,
                                  int32_t *coord, int64_t *posn, int64_t *cost, hipStream_t stream);

// Items one wavefront can stage for SpMV (partition work must not exceed it).
int spmv_capacity(int dtype);
// Non-zeros of a partition of a call that leaves their number to the library (P = 0): the capacity or less.
int64_t spmv_grain(int dtype, int64_t nnz, int64_t n_rows);
// SPMV_TABLE: any partition table; SPMV_DEALT: the table of the fixed-grain queries Q_p = min(p * grain, nnz), dealt out by
// XCD inside long rows; SPMV_SEARCH: no table, every wavefront searches its own boundaries (y has been cleared);
// SPMV_WHOLE: the same, and the kernel writes the table and the zeros of empty rows itself.
enum SpmvForm { SPMV_TABLE = 0, SPMV_DEALT = 1, SPMV_SEARCH = 2, SPMV_WHOLE = 3 };
// Whether a fixed-grain call with P partitions takes the last form.
bool spmv_whole(int dtype, int64_t nnz, int64_t grain, int64_t P, int64_t n_rows, int64_t x_bytes);
hipError_t launch_spmv_exec(int dtype, const int32_t *pos, const int32_t *crd, const void *val,
                            const void *x, void *y, int64_t n_rows, int64_t nnz,
                            int32_t *coord, int32_t *posn, int64_t *cost, int64_t P,
                            void *carry_val, int32_t *carry_row, int64_t grain, SpmvForm form, hipStream_t stream);
hipError_t launch_zero_vector(int dtype, void *y, int64_t n, hipStream_t stream);
hipError_t launch_spmv_fixup(int dtype, void *y, int64_t P, const void *carry_val,
                             const int32_t *carry_row, const int32_t *pos, int64_t grain, hipStream_t stream);

// ---- SpMM ------------------------------------------------------------------
int spmm_capacity();                                // most non-zeros of a partition
// Whether a fixed-grain call sorts its partitions by column (row_bytes: of a row of B).
bool spmm_dealt(int64_t nnz, int64_t n_cols, int64_t row_bytes);
int spmm_grain(int64_t nnz, int units, bool dealt, int64_t row_bytes);      // non-zeros of a fixed-grain partition
// Whether a fixed-grain call goes without a partition kernel (the executing kernel writes the table and the zeros).
bool spmm_whole(int64_t P, int64_t n_rows);
// Workgroup w executes partition sorted[place[w]], or partition w where place[w] is -1.  Where all of them are -2, the workgroups
// w < joined execute partitions w * join .. of the table in one piece.  NULL: workgroup w partition w.
struct SpmmDeal {
    int32_t *place, *sorted;
    int join, joined;
};
int64_t spmm_deal_words(int64_t P);                 // 32-bit words it takes
// row_bytes: of a row of B in one pass.  join: partitions that make up one of an unsorted call (1: they are never joined).
hipError_t launch_spmm_deal(const int32_t *coord, int64_t P, int64_t n_cols, int64_t row_bytes, int join, int32_t *words,
                            SpmmDeal *deal, hipStream_t stream);
// carry_val: n values per partition.  b_bytes: of B.  `grain` (non-zeros) > 0: fixed-grain partitions.
hipError_t launch_spmm_exec(int dtype, const int32_t *pos, const int32_t *crd, const void *val,
                            const void *B, int n, int64_t ldb, void *C, int64_t ldc, int64_t n_rows, int64_t nnz,
                            int32_t *coord, int32_t *posn, int64_t *cost, int64_t P, void *carry_val,
                            int32_t *carry_row, int64_t grain, int64_t cost_scale, bool whole, const SpmmDeal &deal,
                            double b_bytes, hipStream_t stream);
hipError_t launch_spmm_fixup(int dtype, void *C, int64_t ldc, int n, int64_t P, const void *carry_val,
                             const int32_t *carry_row, const int32_t *pos, const int32_t *posn, int64_t grain,
                             const SpmmDeal &deal, hipStream_t stream);

// ---- k-way union addition ---------------------------------------------------
enum { SPADD_VECTOR = 0, SPADD_CSR = 1, SPADD_DCSR = 2, SPADD_COO = 3, SPADD_CSF3 = 4 };

struct SpaddValues { const void *v[NACHO_MAX_OPERANDS]; };
struct SpaddOut {
    int32_t *pos0, *crd0, *pos1, *crd1;
    void *val;
    int64_t cap_rows, cap_nnz;
    int32_t *pos2, *crd2;        // third-order tensors: the innermost level (crd1 / pos2: the fibres)
    int64_t cap_fibres;
    int64_t *counts;
    int32_t *status;
};
// Partitions of a merge that needs `need` of them, on a chip that holds `round` of its workgroups at a time: a whole
// number of rounds where that adds a twelfth at most, else as few as will do.  Workgroups come and go one by one, so a last
// round need not be full; shorter partitions pay a partition's fixed time more often.  Measured on sums of vectors, CSR
// matrices, coordinate lists, DCSR matrices and tensors with 3 to 16 % more partitions than needed (whole rounds against
// as few as will do): one and two rounds of matrices and tensors -5 to +1 % up to 13 % more, -5 to +4 % at 16 %; four
// rounds -2 to 0 % at 3 and 6 %, -1 to +2 % at 8 %, +0 to +4 % at 10 to 16 %.  Vectors: 0 to +3 % at one and two
// rounds, +3 to +5 % at four.  So the line is a mean: the gains of a few rounds end where the losses of many begin.
__host__ __device__ inline int64_t whole_rounds(int64_t need, int64_t round)
{
    const int64_t up = (need + round - 1) / round * round;
    return (up - need) * 12 <= need ? up : need;
}

// How the merge kernel packs the coordinates of a matrix or tensor entry into a key: row field << cb | column; for a
// tensor the row field is (i - i0) << jb | j.  Rows (slices) count from the partition's first one and a key tells
// `limit` of them apart.  `wide`: 64-bit keys.  `size`: how many places of the merged order a thread owns (MergeSize).
enum MergeSize : int { MERGE_LONG, MERGE_SHORT, MERGE_MIDDLE };
// `touch`: the lines of the values are asked for beside the merge (kernels that can).
struct MergeFields {
    int32_t cb, jb, wide, size;
    uint32_t limit;
    int32_t touch;
};
// `k` operands; `rows`, `cols`, `depth`: the extents of the levels; `total`: stored entries of all operands; `units`: compute units;
// `mapped`: remapped operands.
MergeFields merge_fields(int fmt, int dtype, int k, int64_t rows, int64_t cols, int64_t depth, int64_t total, int units,
                         bool mapped = false);
// Entries of all operands one partition (workgroup) may hold.
int spadd_capacity(int fmt, int dtype, const MergeFields &fields);
// Workgroups of the merge kernel that run on one compute unit at a time.
int spadd_resident();
// Wavefronts of one of its workgroups (the instrumented build logs one record per wavefront).
int spadd_wavefronts();
// 64-bit words of prefix-sum state a call with P partitions uses.
int64_t spadd_state_words(int64_t P);
// The partition table a merge kernel that searches its own boundaries fills, and the total cost Q*.
struct SpaddSearch {
    int32_t *coord, *posn;
    int64_t *cost;
    int64_t total;
};
// Sparse vectors, union: as launch_spadd, but without a partition kernel before it -- every workgroup
// searches its two boundaries (equal-share queries over P partitions) and stores them in the table.
// The prefix-sum state and the status word must be zero when the kernel starts.
hipError_t launch_spadd_vector_search(int dtype, const DevOperands &ops, const SpaddValues &vals, int64_t P,
                                      const SpaddSearch &search, unsigned long long *tile_state, const SpaddOut &out,
                                      const MergeFields &fields, hipStream_t s);
// Count, prefix sum and fill in one kernel, one workgroup per partition.  `multiply`: the k-way
// intersection with products instead of the union with sums (vectors, CSR and coordinate lists; DCSR operands come
// here remapped, as CSR; no tensors).
hipError_t launch_spadd(int fmt, int dtype, bool multiply, const DevOperands &ops, const SpaddValues &vals,
                        int64_t P, const int32_t *coord, const int32_t *posn, unsigned long long *tile_state,
                        const SpaddOut &out, const MergeFields &fields, hipStream_t s);

// The merge kernel's instantiations, one translation unit per format.
struct MergeLaunch {
    const DevOperands &ops;
    const SpaddValues &vals;
    int64_t P;
    const int32_t *coord, *posn;
    unsigned long long *tile_state;
    const SpaddOut &out;
    MergeFields fields;
    SpaddSearch search;
    hipStream_t s;
};
hipError_t merge_vector(int dtype, bool multiply, const MergeLaunch &a);
hipError_t merge_vector_search(int dtype, const MergeLaunch &a);
hipError_t merge_csr(int dtype, const MergeLaunch &a);
hipError_t merge_csr_product(int dtype, const MergeLaunch &a);
hipError_t merge_csr_mapped(int dtype, const MergeLaunch &a);
hipError_t merge_dcsr(int dtype, const MergeLaunch &a);
hipError_t merge_coo(int dtype, bool multiply, const MergeLaunch &a);
hipError_t merge_csf3(int dtype, const MergeLaunch &a);

// ---- recursive partitioning for an outer intersection (DCSR products) -----------
// Memoised row loop of Section 3.3, all arrays on the device:
//   rows[i']                    coordinate of the i'-th row all operands store
//   start[t * stride + i']      position in operand t's crd / val of that row's first entry
//   cost[t * (stride + 1) + x]  entries operand t stores in the intersected rows before row x (x <= M)
//   head[0] = number M <= stride of intersected rows, head[1 + t] = cost[t][M]
struct RemapArrays {
    int32_t *rows, *start, *cost, *head;
    int64_t stride;
};
constexpr int kRemapGrain = 1024;      // level-0 coordinates of all operands per partition of the row loop
// 64-bit words of look-up state, zero when the kernel starts.
int64_t remap_state_words(int64_t P0, int k);
int64_t compact_state_words(int64_t rows);
// The row loop.  posn0: boundaries of a P0-way partition of the operands' level-0 coordinate arrays.  Also
// plan[0..2] = {partitions of the remapped nest, intersected rows, remapped total cost}: capacity = entries one
// partition may hold, round = resident workgroups of the chip (the count is rounded up to whole rounds when
// P_min == 0), P_max = what the launches are sized for.  plan[3], zero when the kernel starts, is set when a
// workgroup's wait ran out: the kernels behind it then leave at once, *status is NACHO_ERR_HIP.
hipError_t launch_remap_rows(const DevOperands &ops, int64_t P0, const int32_t *posn0, const RemapArrays &r,
                             unsigned long long *state, int64_t capacity, int64_t round, int64_t P_min, int64_t P_max,
                             int64_t *plan, int32_t *status, hipStream_t s);
// Result rows that hold an entry: pos_full[0 .. head[0]] over the intersected rows -> out.pos0 / crd0 /
// pos1 / counts (counts_in = {rows, nnz} of the remapped result).
hipError_t launch_compact_rows(const RemapArrays &r, const int32_t *pos_full, const int64_t *counts_in,
                               const int64_t *plan, const SpaddOut &out, unsigned long long *state, hipStream_t s);
hipError_t launch_empty_result(const SpaddOut &out, int64_t *info, hipStream_t s);

// ---- measurement aids: kernels of known traffic (streaming read, copy, independent gathers) ----
hipError_t launch_probe_read(const void *src, size_t bytes, void *sink, hipStream_t s);
hipError_t launch_probe_copy(void *dst, const void *src, size_t bytes, hipStream_t s);
hipError_t launch_probe_gather(const void *table, size_t window_bytes, int64_t gathers, void *sink, hipStream_t s);

// ---- debug aid: the preconditions of the operands, checked on the device -----------
hipError_t launch_validate(const DevOperands &ops, int32_t *status, int64_t *info, hipStream_t s);

}  // namespace nacho
