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

int capacity_of(bool wide, int size, int dtype)
{
    if (wide) return dtype == NACHO_F64 ? Shape<uint64_t, double, MERGE_LONG>::kCapacity : Shape<uint64_t, float, MERGE_LONG>::kCapacity;
    if (size == MERGE_SHORT) return dtype == NACHO_F64 ? Shape<uint32_t, double, MERGE_SHORT>::kCapacity : Shape<uint32_t, float, MERGE_SHORT>::kCapacity;
    if (size == MERGE_MIDDLE) return dtype == NACHO_F64 ? Shape<uint32_t, double, MERGE_MIDDLE>::kCapacity : Shape<uint32_t, float, MERGE_MIDDLE>::kCapacity;
    return dtype == NACHO_F64 ? Shape<uint32_t, double, MERGE_LONG>::kCapacity : Shape<uint32_t, float, MERGE_LONG>::kCapacity;
}

}  // namespace

// Workgroups of the merge kernel a compute unit holds at a time (its LDS and registers are cut for that).
int spadd_resident() { return 32 / kWaves; }
int spadd_wavefronts() { return kWaves; }

// The key layout of a call: 32-bit keys when the rows (slices) that an average full partition spans take a
// quarter of the row field or less, or the field holds any row, else 64-bit keys.  A partition that spans more rows
// than the field holds is merged by searches (rank_far), for which a key's word has to hold any (slice, fibre) pair.
MergeFields merge_fields(int fmt, int dtype, int k, int64_t rows, int64_t cols, int64_t depth, int64_t total, int units, bool mapped)
{
    MergeFields f;
    f.cb = f.jb = f.wide = f.touch = 0;
    f.limit = 0;
    // Short partitions while two of them a compute unit hold a call (vectors; CSR, 16 entries a row and more), a whole round of them (other CSR; five
    // and more coordinate lists) or five sixths of one (the others), middle ones while one round of workgroups does, else long ones.  A partition
    // takes some 8 us whatever it holds, so few long ones beat many short ones; but a thread's serial share is what a round takes, so no longer
    // than need be.  Sums of two vectors, CSR matrices, tensors of 32-bit values, us: 700k entries in all, short 14.2, 16.9, 24.2, middle 13.5, 16.7,
    // 24.9; 1.1M 16.1, 20.3, 27.6 and 14.4, 18.1, 27.9; 1.45M 17.8, 22.7, 30.8 and 15.7, 20.6, 29.0; 3M, long 21.4, 25.8, 39.3, middle 19.9, 24.9, 35.1.
    // DCSR matrices with three entries a row, two and four operands, 1M short 26.7, 40.5, middle 27.2, 44.1; 1.4M 33.0, 47.5 and 31.8, 46.2; CSR with four
    // 1M 22.8, 32.4 and 24.2, 35.4, 1.4M 26.1, 36.7 and 26.3, 37.2; coordinate lists, four, five, eight operands, 1.4M to 1.5M 39.5, 49.4, 61.5 and 39.4, 51.7,
    // 64.5.  Products of 700k take 1.04 to 1.08 of the time as middle ones, of 900k 0.96 to 1.04.
    auto fits = [&](int size, double per_unit) {       // (workgroups on a compute unit)
        return (double)total <= (double)units * per_unit * (double)(capacity_of(false, size, dtype) - NACHO_MAX_OPERANDS);
    };
    const int resident = spadd_resident();
    double short_ones = 5.0 * resident / 6.0;
    if (fmt == SPADD_VECTOR || (fmt == SPADD_CSR && total >= 16 * rows)) short_ones = resident / 2;
    else if (fmt == SPADD_CSR || (fmt == SPADD_COO && k > 4)) short_ones = resident;
    // (remapped operands: the total counts entries that are not coiterated)
    if (fits(MERGE_SHORT, mapped ? resident : short_ones)) f.size = MERGE_SHORT;
    else if (mapped) f.size = MERGE_MIDDLE;
    // (doubles of vectors and tensors have ten places a thread only where one round of them holds a call that one of nine does not: 4.7M entries,
    // vectors of two, three, eight operands 24.2, 36.5, 59.3 us and 27.1, 40.0, 62.4 with nine, tensors 62.9, 73.3, 99.7 and 68.7, 81.6, 116.9; past that
    // round, 5.3M, 28.7, 42.4, 68.4 and 27.8, 44.4, 64.2, tensors 75.5, 90.0, 127.6 and 73.2, 87.5, 120.8, of 8M 47.0, 58.3, 87.1 and 46.5, 58.4,
    // 84.4, tensors 85.9, 103.1, 145.7 and 82.9, 98.5, 136.2.  Matrices keep ten: 5.3M CSR 33.4, 46.6, 71.6 and 36.4, 47.7, 72.4, DCSR 39.6, 46.9, 73.7
    // and 40.6, 51.0, 76.5, lists 47.5, 57.6, 92.4 and 49.9, 63.1, 95.9; of 8M equal within 2 %)
    else if (!fits(MERGE_MIDDLE, resident))
        f.size = dtype == NACHO_F64 && (fmt == SPADD_VECTOR || fmt == SPADD_CSF3) && !fits(MERGE_LONG, resident) ? MERGE_MIDDLE : MERGE_LONG;
    // two long partitions a compute unit instead of three middle ones (2.6M entries, two and eight operands, us: CSR 23.2 and 23.6, 48.9 and 50.7; DCSR
    // 27.8 and 28.1, 54.9 and 58.0; but vectors 19.3 and 19.1, 46.4 and 46.7, tensors 35.2 and 33.9, 61.5 and 60.9)
    else if ((fmt == SPADD_CSR || fmt == SPADD_DCSR) && dtype == NACHO_F32 && !fits(MERGE_MIDDLE, 2) && fits(MERGE_LONG, 2)) f.size = MERGE_LONG;
    else f.size = MERGE_MIDDLE;
    if (fmt == SPADD_VECTOR) return f;
    // Values asked for ahead: coordinate lists past what short partitions hold (some 1.25M entries, whatever the keys) and tensors past a few
    // million, whose values come from memory itself and whose partitions ask for little else beside their merge.  us without and with it, the
    // same operands again and operands that no cache holds: two lists of floats, 1.6M 22.2, 22.2 and 26.2, 25.8, 2.5M 25.9, 25.2 and 29.7, 29.1,
    // 4.5M 33.0, 33.1 and 40.1, 37.4; of doubles 23.6, 23.7 and 27.7, 27.4, 27.4, 27.3 and 32.5, 31.7, 35.5, 35.1 and 45.2, 41.5; three of
    // doubles 37.5, 37.6 and 39.3, 39.1, 39.4, 39.3 and 45.6, 43.7, 49.2, 49.2 and 57.7, 54.6 (of floats the same but for 3 %).  The same operands
    // again, two lists of floats, 5M, 6M, 8M, 20M 37.0, 42.0, 57.3, 120.7 and 34.4, 37.1, 54.2, 117.9; of doubles, 6M, 20M 55.4, 144.9 and 51.2, 144.3;
    // three of doubles, 5M, 12M, 35M 0.91, 0.98 and 1.02 of the time; two tensors of floats, 2.5M, 4.5M, 6M, 35M 0.99, 0.95, 0.96, 0.97, of
    // doubles, 1.5M, 4.5M, 12M 1.04, 0.93, 1.00; three 1.01, 0.95, 1.02.  Not five (1.01), products, which ask for few, or other formats (two
    // vectors of doubles, 5M 1.10, two CSR matrices, 20M 1.07: their values' lines leave the L2s again before the places ask for them).
    if (fmt == SPADD_COO) f.touch = !fits(MERGE_SHORT, short_ones) && (k == 2 || (k == 3 && total <= 14'000'000));
    else if (fmt == SPADD_CSF3 && total >= 3'200'000)
        f.touch = dtype == NACHO_F32 ? k == 2 : (k <= 3 && fits(MERGE_LONG, resident));
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
    auto needs_wide = [&](int size) {
        int64_t span = (int64_t)((double)rows * capacity_of(false, size, dtype) / (double)per) + 2;
        if (span > rows) span = rows;
        return f.limit == 0 || (fmt == SPADD_CSF3 && rows > (int64_t)1 << (32 - f.jb)) ||
               (rows > (int64_t)f.limit && span > (int64_t)(f.limit / 4));
    };
    // Tensors whose middle partitions would need 64-bit keys stay with short ones of 32-bit keys as long as those are one round (two, three,
    // five of 1.3M entries in all, 2000 x 2000 x 2000, us: 31.3, 37.5, 48.0 and 33.7, 42.3, 52.9 with 64-bit keys).  Matrices do not (DCSR,
    // coordinate lists of 1.4M, 400,000 rows, 1M columns, short against 64-bit keys: 31.7 and 29.9, 24.9 and 21.6).
    if (fmt == SPADD_CSF3 && f.size == MERGE_MIDDLE && fits(MERGE_SHORT, resident) && needs_wide(MERGE_MIDDLE) && !needs_wide(MERGE_SHORT))
        f.size = MERGE_SHORT;
    if (needs_wide(f.size)) {
        f.wide = 1;
        f.size = MERGE_LONG;
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

int spadd_capacity(int fmt, int dtype, const MergeFields &f) { (void)fmt; return capacity_of(f.wide != 0, f.size, dtype); }

// 64-bit words of look-up state: one per chunk, then one 32-bit word per workgroup -- twice (third-order
// tensors count slices in the second set); sized for the smallest chunk, which covers all
int64_t spadd_state_words(int64_t P) { return 2 * (chunks_of(P, kChunkProduct) + (P + 1) / 2); }

hipError_t launch_spadd_vector_search(int dtype, const DevOperands &ops, const SpaddValues &vals, int64_t P,
                                      const SpaddSearch &search, unsigned long long *tile_state, const SpaddOut &out,
                                      const MergeFields &fields, hipStream_t s)
{
    const MergeLaunch a{ops, vals, P, search.coord, search.posn, tile_state, out, fields, search, s};
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
