// The boundary search of Algorithm 1 (Section 3.2) as one wavefront runs it, for the partition
// kernel and for kernels that search their own boundaries: see partition.hip for the method.
#pragma once
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"

namespace nacho {

namespace {

// How a compressed level's coordinates are read.  Plain: one int32 array.  Pairs: the level is
// the list of (row, column) pairs of a coordinate-list (COO) operand, i.e. both of its levels
// taken together as one sorted, duplicate-free level with the 64-bit coordinate row << 32 | column
// (Algorithm 1 on the two levels and on this one level find the same boundary: the highest row
// whose cost fits, then the highest column inside it, is the highest pair whose cost fits).
typedef const __attribute__((address_space(1))) int32_t *Ints32;
__device__ inline Ints32 as_global(const int32_t *a) { return (Ints32)(unsigned long long)(uintptr_t)a; }

struct PlainCoords {
    typedef int type;
    static constexpr bool kPairs = false;
    static constexpr type kNone = INT32_MAX;            // no coordinate
    Ints32 crd;
    __device__ type load(int at) const { return crd[at]; }
    __device__ static PlainCoords of(const DevOperands &ops, int t, int m) { return PlainCoords{as_global(ops.lvl[t][m].crd)}; }
    __device__ static int64_t extent(const DevOperands &ops, int m) { return ops.lvl[0][m].extent; }
};
struct PairCoords {
    typedef long long type;
    static constexpr bool kPairs = true;
    static constexpr type kNone = INT64_MAX;
    Ints32 row, col;
    __device__ type load(int at) const { return ((long long)row[at] << 32) | (long long)(unsigned)col[at]; }
    __device__ static PairCoords of(const DevOperands &ops, int t, int)
    {
        return PairCoords{as_global(ops.lvl[t][0].crd), as_global(ops.lvl[t][1].crd)};
    }
    __device__ static int64_t extent(const DevOperands &ops, int) { return ops.lvl[0][0].extent << 32; }
};

// Sum, maximum and minimum over the wavefront by DPP moves (in every lane).
__device__ inline int sum_of_lanes(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);    // row_shr:1, 2, 4, 8: inside 16 lanes
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);    // row_bcast:15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);    // row_bcast:31 into rows 2 and 3
    return lane_value(v, NACHO_WAVE - 1);
}
template <int kCtrl, int kRowMask> __device__ inline int moved(int none, int v)
{
    return __builtin_amdgcn_update_dpp(none, v, kCtrl, kRowMask, 0xf, false);
}
template <int kCtrl, int kRowMask> __device__ inline long long moved(long long none, long long v)
{
    const unsigned lo = (unsigned)moved<kCtrl, kRowMask>((int)(unsigned)none, (int)(unsigned)v);
    return ((long long)moved<kCtrl, kRowMask>((int)(none >> 32), (int)(v >> 32)) << 32) | (long long)lo;
}
// `none`: no lane's value comes after it (max) / before it (min).
template <bool kMax, typename C> __device__ inline C extreme_of_lanes(C v, C none)
{
    auto fold = [&](C o) { v = (kMax ? o > v : o < v) ? o : v; };
    fold(moved<0x111, 0xf>(none, v));
    fold(moved<0x112, 0xf>(none, v));
    fold(moved<0x114, 0xf>(none, v));
    fold(moved<0x118, 0xf>(none, v));
    fold(moved<0x142, 0xa>(none, v));
    fold(moved<0x143, 0xc>(none, v));
    return lane_value(v, NACHO_WAVE - 1);
}

// Dense level (level 0 of CSR operands): position == coordinate, cost through
// the next level's pos array.  64-ary search over [0, N].  Returns the row, its cost in c_low, and in first[t], behind[t] where
// operand t's entries of the row start and end (the rounds have looked at both; behind: not of row N).
template <int K>
__device__ __forceinline__ int64_t dense_search(const DevOperands &ops, int64_t R, int64_t &c_low, int (&first)[K], int (&behind)[K])
{
    const int lane = lane_id();
    const int k = ops.k;
    int64_t low = 0, high = level0_extent(ops);
    c_low = 0;
#pragma unroll
    for (int t = 0; t < K; ++t) first[t] = behind[t] = 0;      // (pos[0] = 0)
    while (low < high) {
        const int64_t span = high - low;
        const int64_t step = (span + NACHO_WAVE - 1) / NACHO_WAVE;
        int64_t x = low + (int64_t)(lane + 1) * step;
        if (x > high) x = high;
        int64_t c = 0;
        int at[K];
#pragma unroll
        for (int t = 0; t < K; ++t) {
            at[t] = 0;
            if (t < k) at[t] = ops.lvl[t][1].pos[x];
            c += (int64_t)at[t];
        }
        const unsigned long long ok = __ballot(c <= R);   // a prefix of the lanes (monotone cost)
        const int n = __popcll(ok);
        if (n > 0) {
            low = lane_value((long long)x, n - 1);
            c_low = lane_value((long long)c, n - 1);
#pragma unroll
            for (int t = 0; t < K; ++t) first[t] = lane_value(at[t], n - 1);
        }
        if (n < NACHO_WAVE) {
            high = lane_value((long long)x, n) - 1;
#pragma unroll
            for (int t = 0; t < K; ++t) behind[t] = lane_value(at[t], n);
        }
    }
    return low;
}

// ---- compressed levels ---------------------------------------------------------
// The lanes of a wavefront are split into k groups of 64 / k, one operand each: lane i of a group holds that operand's
// window, and its i-th sample of it.  What bounds a search is the chain of rounds -- a load each, and some 300 instructions
// -- and, with thousands of boundaries in flight, the cache lines it asks for.  (A lane for one of 64 samples of EVERY
// operand asks for k times the lines, keeps k times the state, and has k (k - 1) ranks to find instead of k - 1: three
// operands of 10M, 1M and 100k entries 19.2 us, like this 12.8; with that many operands that it searched coordinates instead, with
// binary searches inside: five vectors of 2.5M 119 and 21.7, eight coordinate lists of 1.4M 256 and 65, eight tensors
// of 1M 100 and 30.)
template <int K> struct Group {
    int k, size;               // groups, lanes of one
    int t, i, first;           // this lane's group, its place in it, the group's first lane (a lane left over: i >= size)
    unsigned long long lanes;  // of the group
    __device__ explicit Group(int k_) : k(k_)
    {
        const int lane = lane_id();
        size = NACHO_WAVE;                     // (64 / k without a division)
        if (K > 1) size = k == 1 ? 64 : (k == 2 ? 32 : (k == 3 ? 21 : 16));
        if (K > 4 && k > 4) size = k == 5 ? 12 : (k == 6 ? 10 : (k == 7 ? 9 : 8));
        t = 0;
#pragma unroll
        for (int u = 1; u < K; ++u) t += (u < k ? 1 : 0) & (lane >= u * size ? 1 : 0);
        first = t * size;
        i = lane - first;
        lanes = low_bits(first + size) & ~low_bits(first);
    }
    // the value the group's lane `at` holds
    template <typename C> __device__ C from(C v, int at) const { return value_from(v, first + at); }
    __device__ int count(unsigned long long mask) const { return __popcll(mask & lanes); }
    __device__ bool any(unsigned long long mask) const { return (mask & lanes) != 0ull; }
    // sum of the groups' values (the same in all lanes of a group)
    __device__ int sum(int v) const
    {
        if (K > 4) return sum_of_lanes(i == 0 ? v : 0);
        int x = lane_value(v, 0);
#pragma unroll
        for (int u = 1; u < K; ++u)
            if (u < k) x += lane_value(v, u * size);
        return x;
    }
};

// How many of the `size` values of the group that starts at lane b -- ascending, the ones past the valid ones hold the
// largest value there is -- are smaller than this lane's key.  Four ways a step: two or three dependent shuffles.
template <int K, typename C> __device__ inline int rank_in(C v, int b, int size, C key)
{
    int c = 0;
    auto step = [&](auto ways_tag, auto stride_tag) {
        constexpr int kWays = decltype(ways_tag)::value, kStride = decltype(stride_tag)::value;
        C x[kWays];
#pragma unroll
        for (int g = 0; g < kWays; ++g) {
            const int at = c + (g + 1) * kStride;
            x[g] = value_from(v, b + (at < size ? at : size) - 1);
        }
        int more = 0;
#pragma unroll
        for (int g = 0; g < kWays; ++g) more += c + (g + 1) * kStride <= size && x[g] < key ? 1 : 0;
        c += more * kStride;
    };
    typedef std::integral_constant<int, 1> One;
    typedef std::integral_constant<int, 2> Two;
    typedef std::integral_constant<int, 3> Three;
    if constexpr (K <= 2) {                    // up to 32
        step(Two(), std::integral_constant<int, 16>());
        step(Three(), std::integral_constant<int, 4>());
        step(Three(), One());
    } else if constexpr (K <= 4) {             // up to 21
        step(Two(), std::integral_constant<int, 8>());
        step(Three(), Two());
        step(One(), One());
    } else {                                   // up to 12; two ways a step: the other groups' searches hide each other
        step(One(), std::integral_constant<int, 8>());
        step(One(), std::integral_constant<int, 4>());
        step(One(), Two());
        step(One(), One());
    }
    return c;
}

// Where sample i of `size` lies in a window of w > size entries when the coordinate is expected `at` entries in: the
// window's ends are samples, the others lie at distances from `at` that grow geometrically, from half the deviation that
// positions have when the operands' entries are spread alike (at most sqrt(w) / 4) to the window's ends.  An
// expectation that is off by e leaves a window of about e; entries that are spread alike (the columns of a row, the
// coordinates of a vector) go from ten million to a few thousand to under a hundred.  `even`: evenly spaced.
__device__ inline int aimed_sample(int i, int size, int w, float at, bool even)
{
    // (the reciprocals need not be exact: any place in the window will do)
    const float inv = 2.0f * __builtin_amdgcn_rcpf((float)(size - 1)), all = (float)w;
    const float e = (float)i * inv - 1.0f;             // -1 .. 1
    float x = 0.5f * (all + all * e);
    if (!even) {
        const float left = fmaxf(at, 1.0f), right = fmaxf(all - at, 1.0f);
        const float near = fmaxf(0.5f * __builtin_amdgcn_sqrtf(left * right * __builtin_amdgcn_rcpf(left + right)), 0.5f);
        const float side = fmaxf(e < 0.0f ? left : right, near);
        const float off = near * __builtin_amdgcn_exp2f(fabsf(e) * __builtin_amdgcn_logf(side * __builtin_amdgcn_rcpf(near)));
        x = fabsf(e) * (float)size < 0.5f ? at : at + copysignf(off, e);
    }
    int s = (int)fminf(fmaxf(x, 0.0f), fminf(all, 2147483520.0f));
    s = s < w - 1 ? s : w - 1;
    return i == 0 ? 0 : (i == size - 1 ? w - 1 : s);
}

// The first position in [a, z) of the group's operand that is not `before` what is looked for, z if all are: the probes of
// a round are spread evenly over the group's lanes, those before it are a prefix of them.
template <int K, class Before> __device__ inline int group_lower_bound(const Group<K> &g, int a, int z, Before &&before)
{
    while (__ballot(a < z) != 0ull) {
        // (unsigned: probes behind z may lie past 2^31)
        const unsigned stride = (unsigned)(z - a + g.size - 1) / (unsigned)g.size, from = (unsigned)a;
        const unsigned probe = from + (unsigned)(g.i + 1) * stride - 1u;
        const bool yes = g.i < g.size && a < z && probe < (unsigned)z && before((int)probe);
        const unsigned m = (unsigned)g.count(__ballot(yes));
        if (a < z) {
            const unsigned a_new = from + m * stride, z_new = from + (m + 1u) * stride - 1u;
            z = m < (unsigned)g.size && z_new < (unsigned)z ? (int)z_new : z;
            a = a_new < (unsigned)z ? (int)a_new : z;
        }
    }
    return a;
}

// What a level's search finds.
template <class Acc> struct LevelFound {
    typename Acc::type x;      // the boundary's coordinate
    int c;                     // cost of the level's entries before it
    // in the lanes of every group:
    int p;                     // the operand's first entry that is not before x
    bool present;              // ... is at x
    int lo, hi;                // (not on the last level) the entry's segment one level down, empty if it is not at x
    int deep_lo, deep_hi;      // (kDepth 2) its segment two levels down
    int row_from;              // (pairs) no entry of x's row lies before this position
};

// A compressed level.  kDepth: 0 on the last level, where an entry costs 1; 1 where it costs the entries of its segment one
// level down (pos_1); 2 those two levels down (pos_1, then pos_2).  [l, h): the operand's entries of the level, in
// the lanes of its group; `total` their cost, all operands together; 0 <= R < total, so the boundary is a
// stored coordinate.  sh: what is added to positions where coordinates are read (a remapped operand's row).
//
// Invariant: the boundary coordinate x and x + 1 have their positions in [l, h] in every operand.  A round looks at the
// samples of every window.  A sample's position is exact in its own operand; in the others it lies between the two samples
// around it, which bounds its cost from both sides.  The largest sample whose cost is at most R for sure, and the smallest
// whose cost is above it for sure, cut every window.  Once a window has no more entries than its group has lanes every entry is
// a sample; when that holds for all, the costs are exact and the round returns the boundary.
// A round that does not narrow the windows to a half (data that is nothing like evenly spread) is followed by
// one with evenly spaced samples, and if that does not narrow them to three quarters, by one that looks up the exact
// cost of the middle entry of the largest window and so halves that one: the search ends for any operands.
// (Evenly spaced samples leave about four of the size - 1 gaps, 4/7 of the windows with eight lanes: for sorted operands the
// look-up is a safeguard that no spread tried has needed.  Three rounds take a sixteenth off all windows together in the worst
// case: 2^31 entries in 8 operands take a thousand.)
constexpr int kMostRounds = 1100;

// kExact: as search_boundary.
template <int K, class Acc, int kDepth, bool kExact>
__device__ __forceinline__ LevelFound<Acc> group_search(const Group<K> &g, const Acc &crd, Ints32 pos_1, Ints32 pos_2, int l,
                                                        int h, int R, int total, int sh)
{
    typedef typename Acc::type C;
    constexpr bool kLast = kDepth == 0;
    LevelFound<Acc> found;
    // what an entry's position stands for: the cost before it, not yet relative to the segment's start
    auto cost_from = [&](int q, int &below) -> int {
        if (kLast) return below = q;
        below = pos_1[q];
        return kDepth == 2 ? pos_2[below] : below;
    };
    int below_l = l, unused = 0;               // (kDepth 2) pos_1 of l
    int base = cost_from(l, below_l), cl = base, ch = cost_from(h, unused);
    int row_from = l;
    int W = g.sum(h - l);
    float share = (float)R * __builtin_amdgcn_rcpf((float)total);      // of the windows' cost that lies before the boundary
    bool even = false;
    for (int round = 0;; ++round) {
        const int w = h - l, n = w < g.size ? w : g.size;
        const bool small = __ballot(w > g.size && g.i < g.size) == 0ull;
        const bool valid = g.i < n;
        int s = g.i;
        if (!small) {
            const bool wide = w > g.size && valid;
            if (wide) s = aimed_sample(g.i, g.size, w, share * (float)w, even);
            if (__ballot(wide && g.i > 0 && s < lane_left(s)) != 0ull) {      // (rounding: samples have to ascend)
                if (wide) s = aimed_sample(g.i, g.size, w, 0.0f, true);
            }
        }
        s = valid ? l + s : h;
        C v = Acc::kNone;
        int cb, ca, below_b = 0, below_a = 0;  // cost before and behind the sample
        if (valid) v = crd.load(s + sh);
        if (kLast) { cb = s; ca = valid ? s + 1 : s; }
        else {
            cb = ca = 0;
            if (valid) {
                cb = cost_from(s, below_b);
                ca = cost_from(s + 1, below_a);
            }
            cb = valid ? cb : ch;
            ca = valid ? ca : ch;
        }
        // bounds of the sample's cost (no branches: the searches in the other groups hide each other's latency)
        int lo_cost = cb - base, hi_cost = lo_cost;
        int c[K], b[K];
#pragma unroll
        for (int r = 1; r < K; ++r) {
            b[r] = g.first + r * g.size;       // the first lane of another group
            b[r] = g.t + r >= g.k ? b[r] - g.k * g.size : b[r];
            b[r] = r < g.k ? b[r] : g.first;
            c[r] = rank_in<K>(v, b[r], g.size, v);
        }
#pragma unroll
        for (int r = 1; r < K; ++r) {
            // (the first sample is the window's first entry, the last sample of a full group its last one)
            const int before = value_from(ca - base, b[r] + (c[r] > 0 ? c[r] - 1 : 0));
            const int after = value_from(cb - base, b[r] + (c[r] < g.size ? c[r] : g.size - 1));
            lo_cost += r >= g.k ? 0 : (c[r] == 0 ? after : before);
            hi_cost += r >= g.k ? 0 : (c[r] == g.size ? before : after);
        }
        const C none_below = C(-1), none_above = Acc::kNone;
        const unsigned long long surely_before = __ballot(valid && hi_cost <= R), surely_behind = __ballot(valid && lo_cost > R);
        C vminus = none_below, vplus = none_above;
        if constexpr (kExact) {
            // (the bounds ascend with the samples: the last lane of a group, the first one; by a reduction over all lanes two DCSR
            // matrices of 15k entries each 12.9 us, like this 12.6, of 20M 152.2 and 150.5)
#pragma unroll
            for (int u = 0; u < K; ++u)
                if (u < g.k) {
                    const unsigned long long in = low_bits((u + 1) * g.size) & ~low_bits(u * g.size);
                    const unsigned long long a = surely_before & in, z = surely_behind & in;
                    const C va = lane_value(v, a ? 63 - __builtin_clzll(a) : 0), vz = lane_value(v, z ? __builtin_ctzll(z) : 0);
                    vminus = a && va > vminus ? va : vminus;
                    vplus = z && vz < vplus ? vz : vplus;
                }
        } else {
            vminus = extreme_of_lanes<true, C>(valid && hi_cost <= R ? v : none_below, none_below);
            vplus = extreme_of_lanes<false, C>(valid && lo_cost > R ? v : none_above, none_above);
        }
        // cut the windows
        const int c1 = g.count(__ballot(valid && v < vminus));
        const bool at_it = g.any(__ballot(valid && v == vminus));
        const int c2 = g.count(__ballot(valid && v < vplus));
        const int i1 = c1 < g.size ? c1 : g.size - 1, i0 = c1 > 0 ? c1 - 1 : 0, i2 = c2 < g.size ? c2 : g.size - 1;
        if constexpr (Acc::kPairs) {
            const int cr = g.count(__ballot(valid && (v >> 32) < (vminus >> 32)));
            const int to = g.from(s, cr > 0 ? cr - 1 : 0) + 1;
            row_from = cr > 0 ? to : row_from;
        }
        const int s1 = g.from(s, i1), s0 = g.from(s, i0) + 1, s2 = g.from(s, i2);
        const int l_new = at_it ? s1 : (c1 > 0 ? s0 : l), h_new = c2 == n ? h : s2;
        int cl_new = l_new, ch_new = h_new;
        if (!kLast) {
            const int e1 = g.from(cb, i1), e0 = g.from(ca, i0), e2 = g.from(cb, i2);
            cl_new = at_it ? e1 : (c1 > 0 ? e0 : cl);
            ch_new = c2 == n ? ch : e2;
        }
        if (kDepth == 2) {
            const int d1 = g.from(below_b, i1), d0 = g.from(below_a, i0);
            below_l = at_it ? d1 : (c1 > 0 ? d0 : below_l);
        }
        if (small) {
            found.x = vminus;
            found.c = g.sum(cl_new - base);
            found.p = l_new;
            found.present = at_it;
            found.row_from = row_from;
            found.lo = found.hi = found.deep_lo = found.deep_hi = 0;
            if (!kLast) {
                const int behind = g.from(ca, i1), below = g.from(below_a, i1);
                found.lo = kDepth == 2 ? below_l : cl_new;
                found.hi = at_it ? (kDepth == 2 ? below : behind) : found.lo;
                found.deep_lo = cl_new;
                found.deep_hi = at_it ? behind : cl_new;
            }
            return found;
        }
        l = l_new; cl = cl_new;
        h = h_new > l_new ? h_new : l_new; ch = ch_new;        // (never below l, but for operands that are not sorted)
        int W_new = g.sum(h - l);
        const bool slow = even ? W_new > W - (W >> 2) : W_new > (W >> 1);
        if (slow && even) {
            // the middle entry of the largest window, looked up in all of them
            const int wide = extreme_of_lanes<true, int>(g.i < g.size ? h - l : -1, -1);
            const int owner = __ffsll((long long)__ballot(g.i < g.size && h - l == wide)) - 1;
            C mid = Acc::kNone;
            if (h > l) mid = crd.load(l + ((h - l) >> 1) + sh);
            mid = lane_value(mid, owner);
            const int a = group_lower_bound<K>(g, l, h, [&](int at) { return crd.load(at + sh) < mid; });
            int below_at = 0;
            const int cost = cost_from(a, below_at);
            if (g.sum(cost - base) <= R) { l = a; cl = cost; below_l = below_at; }
            else { h = a; ch = cost; }
            W_new = g.sum(h - l);
        }
        even = slow && !even;
        share = (float)(R - g.sum(cl - base)) * __builtin_amdgcn_rcpf((float)(kLast ? W_new : g.sum(ch - cl)));
        W = W_new;
        if (round >= kMostRounds) {
            // (operands that are not sorted, which nothing has to come of but an end: some position of the windows)
            found.x = vminus > none_below ? vminus : C(0);
            found.c = R;
            found.p = l;
            found.present = false;
            found.row_from = row_from < l ? row_from : l;
            found.lo = found.hi = kDepth == 2 ? below_l : cl;
            found.deep_lo = found.deep_hi = cl;
            return found;
        }
    }
}

// Two operands on the last level, where the cost is the number of entries: the boundary of query R is the element
// of rank R of the two merged segments, so the search is for the split of the first R merged entries (the first
// operand first on ties) -- i of them from the first operand for the largest i with A[i - 1] <= B[R - i].  Two loads and a
// ballot a round.  Sixteen candidates, placed around the expected split as the samples above are (its first
// expectation: the operands' shares; later ones from how far apart A and B are at the ends of the range); once the
// range is a few cache lines every lane has one, and once there is a lane for every place left the round is the last: what it
// loads is also what the boundary is made of.  (That asked for by itself, two vectors' sums, us: 30k entries 10.2, so 10.0; 1.2M
// 14.3, 14.1; 35M 128, 127.  All 64 lanes in every round of calls of up to 512 boundaries gain nothing: 10.0, 14.7.)
// (10M + 10M entries, 8192 boundaries, evenly spaced candidates: 64 a round 46 us, 16 24, 8 19 -- with thousands of boundaries in
// flight the lines are what takes the time, a line a candidate, with few of them the rounds are.  Two DCSR matrices of 20M, 7218
// boundaries, both levels: 29.2 us with eight evenly spaced ones, 21.0 like this.)  Coordinate lists' candidates stay evenly
// spaced, a line each however often the range is cut: eight of them with more than a thousand boundaries in flight (`many`), else
// sixteen (16 and 8 a round, us: sums of two lists, 512 boundaries 27.1 and 27.7, 861 36.1 and 36.1; products, 1375 46.6 and 45.6,
// 2402 68.9 and 65.7, 4122 106 and 100).
// Requires both segments non-empty and 0 <= R < their total length.
template <class Acc>
__device__ __forceinline__ LevelFound<Acc> split_search(const Group<2> &g, const Acc &A, const Acc &B, int l, int h, int R, int sh,
                                                        bool many)
{
    typedef typename Acc::type C;
    const int lane = lane_id();
    const int a0 = lane_value(l, 0), b0 = lane_value(l, NACHO_WAVE / 2);
    const int na = lane_value(h, 0) - a0, nb = lane_value(h, NACHO_WAVE / 2) - b0;
    const int a_at0 = a0 + lane_value(sh, 0), b_at0 = b0 + lane_value(sh, NACHO_WAVE / 2);     // where the segments are stored
    int lo = R > nb ? R - nb : 0, hi = R < na ? R : na;
    float at = (float)R * (float)na * __builtin_amdgcn_rcpf((float)na + (float)nb) - (float)lo;
    bool even = Acc::kPairs;                           // (rows of unequal length: an expectation is worth nothing, there is none)
    const int share = Acc::kPairs && many ? 3 : 2;     // log2 of the lanes that share a candidate: they read the same words
    while (hi - lo > NACHO_WAVE - 2) {
        const int w = hi - lo;                         // candidates lo + 1 .. hi
        int i;
        if (w <= 256) i = (lane + 1) * ((w + NACHO_WAVE - 1) / NACHO_WAVE);
        else {
            i = 1 + aimed_sample(lane >> share, NACHO_WAVE >> share, w, at, even);
            if (__ballot(lane > 0 && i < lane_left(i)) != 0ull) i = 1 + aimed_sample(lane >> share, NACHO_WAVE >> share, w, at, true);
        }
        i = lo + (i < w ? i : w);
        const int j = R - i;                           // (i <= R, and i >= R - nb: 0 <= j <= nb)
        const C av = A.load(a_at0 + i - 1);
        const C bv = j < nb ? B.load(b_at0 + j) : Acc::kNone;
        const int n = __popcll(__ballot(av <= bv));    // a prefix of the lanes
        const int lo_new = lane_value(i, n > 0 ? n - 1 : 0), hi_new = lane_value(i, n < NACHO_WAVE ? n : NACHO_WAVE - 1);
        if (n > 0) lo = lo_new;
        if (n < NACHO_WAVE) hi = hi_new - 1;
        if constexpr (!Acc::kPairs) {
            const float apart = (float)(bv - av);      // >= 0 for the prefix
            float f = 0.5f;
            if (n > 0 && n < NACHO_WAVE) {
                const float below = __int_as_float(lane_value(__float_as_int(apart), n - 1));
                f = below * __builtin_amdgcn_rcpf(below - __int_as_float(lane_value(__float_as_int(apart), n)));
            }
            even = !even && hi - lo > w >> 3;
            at = f * (float)(hi - lo);
        }
    }
    // The last round: a lane for every place left, lo among them, and one behind; what the boundary is made of is then in the lanes.
    const int place = lo + lane, left = hi - lo;
    C av = Acc::kNone, bv = Acc::kNone;
    if (lane <= left + 1 && place > 0 && place <= na) av = A.load(a_at0 + place - 1);
    if (lane <= left && R - place < nb) bv = B.load(b_at0 + (R - place));
    const int n = __popcll(__ballot(lane == 0 || (lane <= left && av <= bv)));         // (a prefix of the lanes)
    const int i = lo + n - 1, j = R - i;
    const C a_before = lane_value(av, n - 1), a_at = lane_value(av, n), b_at = lane_value(bv, n - 1);
    const C x = a_at < b_at ? a_at : b_at;
    const int la = i - (i > 0 && a_before == x ? 1 : 0);       // (the coordinate's entry of A may lie before the split)
    LevelFound<Acc> found;
    found.x = x;
    found.c = la + j;
    found.p = g.t == 0 ? a0 + la : b0 + j;
    found.present = false;                             // (the last level: nobody asks)
    found.lo = found.hi = found.deep_lo = found.deep_hi = 0;
    found.row_from = l;
    return found;
}

// One level of Algorithm 1 for one query, 0 <= R: as group_search, and what is shorter than that.
template <int K, class Acc, int kDepth, bool kExact>
__device__ __forceinline__ LevelFound<Acc> search_level(const DevOperands &ops, const Group<K> &g, int m, const Acc &crd,
                                                        Ints32 pos_1, Ints32 pos_2, int l, int h, int R, int total, int sh,
                                                        bool many = false)
{
    LevelFound<Acc> found;
    found.row_from = l;
    found.present = false;
    found.lo = found.hi = found.deep_lo = found.deep_hi = 0;
    if (R >= total) {
        // the query reaches past this level's segments (no valid operands' does): the extent is the highest coordinate
        found.x = (typename Acc::type)Acc::extent(ops, m);
        found.c = total;
        found.p = h;
        if (kDepth > 0) found.lo = found.hi = pos_1[h];
        if (kDepth == 2) found.deep_lo = found.deep_hi = pos_2[found.lo];
        return found;
    }
    if constexpr (kDepth == 0) {
        const unsigned long long filled = __ballot(h > l && g.i == 0);
        const int operands = __popcll(filled);
        if (operands <= 1) {
            // one operand with entries in its segment: the residual indexes it
            const int owner = filled ? __ffsll((long long)filled) - 1 : 0;
            found.p = h > l ? l + R : l;               // (R < total: the operand's own entries)
            typename Acc::type v = Acc::kNone;
            if (h > l) v = crd.load(found.p + sh);
            found.x = lane_value(v, owner);
            found.c = R;
            return found;
        }
        if constexpr (K == 2) return split_search<Acc>(g, Acc::of(ops, 0, m), Acc::of(ops, 1, m), l, h, R, sh, many);
    }
    if constexpr (K > 1 || kDepth > 0) found = group_search<K, Acc, kDepth, kExact>(g, crd, pos_1, pos_2, l, h, R, total, sh);
    return found;
}

// One wavefront searches boundary b (0 <= b <= P) and stores its coordinate, positions and cost.
// kMode: 0 = vectors, CSR, DCSR; 1 = coordinate lists; 2 = three compressed levels (CSF).
// found[t] (operands of one level only): operand t's position of the boundary, in every lane.
// kExact: of exactly K operands, else of at most K.  (A merge kernel that searches its own boundaries is not: it has no registers to
// spare for the masks.)
template <int K, int kMode, bool kExact = false>
__device__ inline void search_boundary(const DevOperands &ops, int64_t cost_scale, int64_t P, int64_t grain,
                                                const int64_t *__restrict__ queries, int64_t total_unscaled,
                                                int32_t *__restrict__ coord, int32_t *__restrict__ posn,
                                                int64_t *__restrict__ cost, int64_t b, int (&found)[K])
{
    const int lane = lane_id();
    const int k = kExact ? K : ops.k, d = ops.d;
#pragma unroll
    for (int t = 0; t < K; ++t) found[t] = 0;
    const int64_t total_scaled = total_unscaled * cost_scale;

    int64_t Q = 0;
    if (queries) Q = queries[b];
    else if (grain > 0) Q = b * grain < total_scaled ? b * grain : total_scaled;
    else if (total_scaled < 0x7fffffffLL && P < 0x7fffffffLL) Q = equal_query_short((unsigned)b, (unsigned)total_scaled, (unsigned)P);
    else Q = equal_query(b, total_scaled, P);
    if (Q < 0) Q = 0;
    const int64_t Qu = cost_scale == 1 ? Q : Q / cost_scale;
    const bool interior = b > 0 && b < P && Qu < total_unscaled;
    int32_t *cb = coord + b * d;
    if (!interior) {
        int32_t *pb = posn + b * (int64_t)k * d;
        const bool end = (b != 0);
        if (lane == 0) {
            for (int m = 0; m < d; ++m) cb[m] = 0;
            if (end) cb[0] = (int32_t)level0_extent(ops);
            for (int t = 0; t < k; ++t)
                for (int m = 0; m < d; ++m) {
                    const DevLevel &L = ops.lvl[t][m];
                    int32_t at = 0;
                    if (end) at = (L.kind == NACHO_DENSE) ? (int32_t)L.extent : (int32_t)L.count;
                    if (end && ops.dyn_head) at = m == 0 ? (int32_t)level0_extent(ops) : (int32_t)last_count(ops, t);
                    pb[t * d + m] = at;
                }
            cost[b] = end ? total_scaled : 0;
        }
        if (end && d == 1) {
#pragma unroll
            for (int t = 0; t < K; ++t)
                if (t < k) found[t] = (int)ops.lvl[t][0].count;
        }
        return;
    }

    // Everything about an operand is in the lanes of its group.
    const Group<K> g(k);
    const bool writer = g.i == 0;
    int32_t *pb = posn + (b * (int64_t)k + g.t) * d;
    auto ints_of = [&](auto get) -> Ints32 {
        Ints32 v = as_global(get(0));
#pragma unroll
        for (int u = 1; u < K; ++u) v = g.t == u ? as_global(get(u)) : v;      // (no branches: one round trip)
        return v;
    };
    auto count_of = [&](int m) -> int {
        int v = (int)ops.lvl[0][m].count;
#pragma unroll
        for (int u = 1; u < K; ++u) v = g.t == u ? (int)ops.lvl[u][m].count : v;
        return v;
    };
    auto plain = [&](int m) { return PlainCoords{ints_of([&](int t) { return ops.lvl[t][m].crd; })}; };
    auto pos_of = [&](int m) { return ints_of([&](int t) { return ops.lvl[t][m].pos; }); };
    int R = (int)Qu;
    const int total = (int)total_unscaled;
    if constexpr (kMode == 1) {
        // coordinate lists, d == 2: one search over the (row, column) pairs; the row-level position of an operand is
        // that of its first entry in the boundary's row
        const PairCoords pairs = {ints_of([&](int t) { return ops.lvl[t][0].crd; }), ints_of([&](int t) { return ops.lvl[t][1].crd; })};
        const auto f = search_level<K, PairCoords, 0, kExact>(ops, g, 0, pairs, nullptr, nullptr, 0, count_of(0), R, total, 0, P > 1024);
        R -= f.c;
        const int x0 = (int)(f.x >> 32), x1 = (int)(f.x & 0xffffffffLL);
        const int row_at = group_lower_bound<K>(g, f.row_from, f.p, [&](int at) { return pairs.row[at] < x0; });
        if (writer) {
            pb[0] = row_at;
            pb[1] = f.p;
        }
        if (lane == 0) {
            cb[0] = x0;
            cb[1] = x1;
        }
    } else if constexpr (kMode == 2) {
        // three compressed levels: Algorithm 1 level by level; a level's cost counts the
        // non-zeros below its entries (two pos arrays down at level 0, one at level 1)
        const Ints32 pos1 = pos_of(1), pos2 = pos_of(2);
        const auto f0 = search_level<K, PlainCoords, 2, kExact>(ops, g, 0, plain(0), pos1, pos2, 0, count_of(0), R, total, 0);
        R -= f0.c;
        const auto f1 = search_level<K, PlainCoords, 1, kExact>(ops, g, 1, plain(1), pos2, nullptr, f0.lo, f0.hi, R,
                                                        g.sum(f0.deep_hi - f0.deep_lo), 0);
        R -= f1.c;
        const auto f2 = search_level<K, PlainCoords, 0, kExact>(ops, g, 2, plain(2), nullptr, nullptr, f1.lo, f1.hi, R,
                                                        g.sum(f1.hi - f1.lo), 0);
        R -= f2.c;
        if (writer) {
            pb[0] = f0.p;
            pb[1] = f1.p;
            pb[2] = f2.p;
        }
        if (lane == 0) {
            cb[0] = f0.x;
            cb[1] = f1.x;
            cb[2] = f2.x;
        }
    } else if (d == 1) {
        const auto f = search_level<K, PlainCoords, 0, kExact>(ops, g, 0, plain(0), nullptr, nullptr, 0, count_of(0), R, total, 0);
        R -= f.c;
#pragma unroll
        for (int t = 0; t < K; ++t)
            if (t < k) found[t] = lane_value(f.p, t * g.size);
        if (writer) pb[0] = f.p;
        if (lane == 0) cb[0] = f.x;
    } else {
        const Ints32 pos1 = pos_of(1);
        int x0, p0, lo, hi, sh = 0;
        if (ops.lvl[0][0].kind == NACHO_DENSE) {
            int64_t c = 0;
            int first[K], behind[K];
            const int64_t row = dense_search<K>(ops, R, c, first, behind);
            R -= (int)c;
            x0 = p0 = (int)row;
            const bool present = row < ops.lvl[0][0].extent;
            lo = first[0];
            hi = behind[0];
#pragma unroll
            for (int u = 1; u < K; ++u) {
                lo = g.t == u ? first[u] : lo;
                hi = g.t == u ? behind[u] : hi;
            }
            if (!present) hi = lo;
            if (ops.start[0]) {                        // a remapped operand's row
                const Ints32 start = ints_of([&](int t) { return ops.start[t]; });
                if (present) sh = start[p0] - lo;
            }
        } else {
            const auto f = search_level<K, PlainCoords, 1, kExact>(ops, g, 0, plain(0), pos1, nullptr, 0, count_of(0), R, total, 0);
            R -= f.c;
            x0 = f.x;
            p0 = f.p;
            lo = f.lo;
            hi = f.hi;
        }
        const auto f = search_level<K, PlainCoords, 0, kExact>(ops, g, 1, plain(1), nullptr, nullptr, lo, hi, R, g.sum(hi - lo), sh);
        R -= f.c;
        if (writer) {
            pb[0] = p0;
            pb[1] = f.p;
        }
        if (lane == 0) {
            cb[0] = x0;
            cb[1] = f.x;
        }
    }
    if (lane == 0) cost[b] = (Qu - R) * cost_scale;
}

}  // namespace

}  // namespace nacho
