// Host side of the k-way merge: capacities, key layout, and which instantiation of the kernel (merge.hpp) a
// call runs.
#include <algorithm>

#include "merge.hpp"

namespace nacho {

namespace {

int bits_of(int64_t extent)                    // bits of the largest coordinate below `extent`
{
    int b = 0;
    while (b < 31 && ((int64_t)1 << b) < extent) ++b;
    return b;
}

int capacity_of(bool wide, bool small, int dtype)
{
    if (wide) return dtype == NACHO_F64 ? Shape<uint64_t, double, false>::kCapacity : Shape<uint64_t, float, false>::kCapacity;
    if (small) return dtype == NACHO_F64 ? Shape<uint32_t, double, true>::kCapacity : Shape<uint32_t, float, true>::kCapacity;
    return dtype == NACHO_F64 ? Shape<uint32_t, double, false>::kCapacity : Shape<uint32_t, float, false>::kCapacity;
}

}  // namespace

// Workgroups of the merge kernel a compute unit holds at a time (its LDS and registers are cut for that).
int spadd_resident() { return 32 / kWaves; }
int spadd_wavefronts() { return kWaves; }

// The key layout of a call: 32-bit keys when the rows (slices) that an average full partition spans take a
// quarter of the row field or less, or the field holds any row, else 64-bit keys.  A partition that spans more rows
// than the field holds is merged by searches (rank_far), for which a key's word has to hold any (slice, fibre) pair.
MergeFields merge_fields(int fmt, int dtype, int64_t rows, int64_t cols, int64_t depth, int64_t total, int units)
{
    MergeFields f;
    f.cb = f.jb = f.wide = 0;
    f.limit = 0;
    // Short partitions as long as all of them run at once: beyond that a second round of them takes longer
    // than one round of long ones.
    f.small = total <= (int64_t)units * spadd_resident() * (capacity_of(false, true, dtype) - NACHO_MAX_OPERANDS) ? 1 : 0;
    if (fmt == SPADD_VECTOR) return f;
    const int64_t per = total > 0 ? total : 1;
    if (fmt == SPADD_CSF3) {
        f.cb = bits_of(depth);
        f.jb = bits_of(cols);
        // (a fibre's row field is kept in 16 bits until the keys are formed)
        const int room = 32 - f.cb - f.jb < 16 - f.jb ? 32 - f.cb - f.jb : 16 - f.jb;
        if (room > 0) f.limit = (1u << room) - 1u;
    } else {
        f.cb = bits_of(cols);
        const int room = 32 - f.cb < 16 ? 32 - f.cb : 16;
        f.limit = (1u << room) - 1u;           // (room >= 1)
    }
    int64_t span = (int64_t)((double)rows * capacity_of(false, f.small != 0, dtype) / (double)per) + 2;
    if (span > rows) span = rows;
    if (f.limit == 0 || (fmt == SPADD_CSF3 && rows > (int64_t)1 << (32 - f.jb)) ||
        (rows > (int64_t)f.limit && span > (int64_t)(f.limit / 4))) {
        f.wide = 1;
        f.small = 0;
        f.limit = 0x80000000u;                 // matrices: any row
        if (fmt != SPADD_CSF3) f.cb = 32;
        else {
            // tensors: the row field (i - i0) << jb | j has what is left of the key, kept in 48 bits before (whose
            // upper 16 are never all ones)
            const int room = (64 - f.cb < 48 ? 64 - f.cb : 48) - f.jb;         // (>= 2)
            if (room < 32) f.limit = (uint32_t)(((uint64_t)1 << room) - 1u);
            if (f.jb > 16) f.limit = std::min(f.limit, 0xffffu << (32 - f.jb));
        }
    }
    return f;
}

int spadd_capacity(int fmt, int dtype, const MergeFields &f) { (void)fmt; return capacity_of(f.wide != 0, f.small != 0, dtype); }

// 64-bit words of look-up state: one per chunk, then one 32-bit word per workgroup -- twice (third-order
// tensors count slices in the second set); sized for the smallest chunk, which covers all
int64_t spadd_state_words(int64_t P) { return 2 * (chunks_of(P, kChunkProduct) + (P + 1) / 2); }

hipError_t launch_spadd_vector_search(int dtype, const DevOperands &ops, const SpaddValues &vals, int64_t P,
                                      const SpaddSearch &search, unsigned long long *tile_state, const SpaddOut &out,
                                      hipStream_t s)
{
    const MergeLaunch a{ops, vals, P, search.coord, search.posn, tile_state, out, MergeFields{}, search, s};
    return merge_vector_search(dtype, a);
}

hipError_t launch_spadd(int fmt, int dtype, bool multiply, const DevOperands &ops, const SpaddValues &vals,
                        int64_t P, const int32_t *coord, const int32_t *posn, unsigned long long *tile_state,
                        const SpaddOut &out, const MergeFields &fields, hipStream_t s)
{
    const MergeLaunch a{ops, vals, P, coord, posn, tile_state, out, fields, SpaddSearch{}, s};
    switch (fmt) {
    case SPADD_VECTOR: return merge_vector(dtype, multiply, a);
    case SPADD_COO: return merge_coo(dtype, multiply, a);
    case SPADD_CSR:
        if (!multiply) return merge_csr(dtype, a);
        return ops.start[0] ? merge_csr_mapped(dtype, a) : merge_csr_product(dtype, a);
    case SPADD_DCSR: if (!multiply) return merge_dcsr(dtype, a); break;
    case SPADD_CSF3: if (!multiply) return merge_csf3(dtype, a); break;
    }
    return hipErrorInvalidValue;    // (a DCSR product reaches this kernel as remapped CSR operands)
}

}  // namespace nacho
