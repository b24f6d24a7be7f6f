// Selection through a list: the automatic choice for most calls (make_list_plan has the rules).
//
// selectBin (paper Section 2.3.1) applied to a sample of the row gives a key T that very probably lies at or below the
// k-th key.  ONE sweep over X then does nothing but compare every element with T and append the few that are not below
// it to a list; whenever the list holds at least k elements it contains the k-th key and is the top of the row,
// exactly, so everything that follows (countBin, selectBin, filter, and the order of the output) works on the list.
// Nothing is counted in the sweep, no digit decides what is kept, and the only thing that many workgroups have to
// agree on is T.  The result never depends on the sample: a list that comes out short (the sample misled), or of which more
// than half the row would have to be kept, has the row done again by one workgroup that selects the k-th key from all of X.
//
//   k_list_held     rows of up to 256 KB: one workgroup per row, which holds the row in registers and needs no sample
//   k_list_part     few rows and a small k: several workgroups hold a row and list their stretches' best
//   k_part_finish   ... one workgroup per row puts those in order
//   k_list_row      longer rows, or many: one workgroup per row does all of the following
//   k_list_stream   (short lists, few rows) many workgroups per row, each of which takes the sample and T for itself: X -> list
//   k_list_bound    (the other calls) one workgroup per row: sample, T
//   k_list_sweep    many workgroups per row: X -> list
//   k_list_finish   (short lists) one workgroup per row: the list, best first, is the output
//   k_list_emit     (long lists, unsorted output) many workgroups per row: what lies in better bins than rank k is output as it comes; its bin is a bucket,
//   k_list_scatter  (long lists, sorted) many workgroups per row: the list into buckets of about 2048 ranks each,
//   k_list_buckets  and one workgroup per bucket puts its ranks in order
//
// The last kernel of each of these also does what is normally not there to be done: lists longer than LDS holds, which one workgroup cuts down first, buckets
// too long for one workgroup, which several put in order, and rows whose list was no use, which one workgroup selects anew.  (A clean-up kernel behind it, which found nothing
// to do, took 3 to 4.6 us of every call: 1024 rows of 2^17 bf16 keys, k = 50, 54.3 us, so 49.2; one of 2^24 fp32 keys, k = 256, 33.6 / 31.8; of 2^26, nine in ten equal, k = 2^16, 96.0 / 93.0.)
//
// List entries are 64-bit numbers, distinct within a row, whose descending order is the order of the output: the
// ordered key (direction applied, 16 or 32 bits) above the inverted index (as many bits as n needs).  An entry holds
// all there is to know about an element but a NaN's payload.
//
// Rows with very many elements equal to T (most of the row one value, or enough of it) would make a long list for nothing.  The
// sample shows that; the sweep then keeps only what is better than T and counts the equal elements of every tile, and
// the ones with the lowest positions are read from X again, straight into the output (ties_of_row).
#include "rtopk_kernels.inl"

namespace rtopk {

constexpr u32 kListBins = 4096;                 // bins of a long list's histogram
constexpr int kListStage = 256;                 // staged entries per wave (short lists)
constexpr int kListStageLong = 512;             // ... (long lists)
constexpr int kListBucketBlock = 512;          // threads per workgroup of the buckets' kernel (4096 entries in LDS)
constexpr u32 kListRowTiles = 128;              // tiles of the longest row that one workgroup takes
constexpr u32 kListTies = 16384;                // equal elements from which on they are counted, not listed

// How a sweep deals a row: tiles of four 16-byte vectors per thread (16 elements, or 32 of 16 bits).
constexpr int kLongBlock = 1024;                // threads per workgroup of a long list's sweep (one workgroup per compute unit)
constexpr int kSharedBlock = 512;               // ... of the sweep of few rows
template <int DT, bool LONG, bool NT = false, int V = 4>
using ListSource = KeySource<DT, LONG ? kLongBlock : kGridBlock, V, NT>;
// Vectors of a tile of a long list's sweep.
__device__ __forceinline__ u32 long_unit(const ListPlan& L) { return L.half != 0 ? (u32)kLongBlock * 2u : (u32)kLongBlock * 4u; }

enum : u32 { kListSkip = 0, kListPlain = 1, kListTied = 2 };

// What k_list_bound decides about a row.
struct ListRow {
    u32 mode;      // kListSkip: nothing wanted; kListPlain: list what is >= T; kListTied: list what is > T, count == T
    u32 T;         // key, direction applied
    u32 exact;     // 1: compare keys; 0: compare the element with the number t
    float t;
    u64 lo;        // long lists: see list_bin
    u32 sh;
    u32 split;     // long lists, 1: the bins lie between splitters
};
static_assert(sizeof(ListRow) % 8 == 0, "read by words");
// What became of a row's long list.  A record of its own: the kernel that writes it has workgroups that still read the decision, and a
// wave that found the decision changed would leave the others of its workgroup alone with sums it never wrote.
struct ListDone {
    u32 total;     // entries
    u32 drop;      // the list was no use, the buckets are not filled: why (rtopk_row_trace::redo_why)
    u32 big;       // 1: a bucket has more than one workgroup puts in order
};
constexpr u32 kListDoneOff = 128;
static_assert(sizeof(ListRow) <= kListDoneOff && kListDoneOff + sizeof(ListDone) <= kListMetaBytes, "both lie before the plan's first offset");
// Bits of rtopk_row_trace::redo: the list was no use; it was too long to put in order in LDS; so were some of its buckets.
enum : u32 { kRedoRow = 1, kRedoList = 2, kRedoBuckets = 4 };

// row_shape, in scalar registers (a ragged batch's comes from memory).
template <int DT>
__device__ __forceinline__ RowShape row_shape_scalar(const Params& P, int row) {
    RowShape r = row_shape<KeyOf<DT>::kBytes>(P, row);
    const u64 x = (u64)(uintptr_t)r.x;
    const u32 lo = (u32)__builtin_amdgcn_readfirstlane((u32)x), hi = (u32)__builtin_amdgcn_readfirstlane((u32)(x >> 32));
    r.x = (const char*)(uintptr_t)(((u64)hi << 32) | lo);  // (the builtin's result is signed: no widening of it)
    r.n = __builtin_amdgcn_readfirstlane(r.n);
    r.k = __builtin_amdgcn_readfirstlane(r.k);
    return r;
}

// A row's decision, read into scalar registers (it is the same for every lane, which a load does not know).
__device__ __forceinline__ ListRow list_row_scalar(const ListRow* p) {
    ListRow r;
    constexpr int kWords = sizeof(ListRow) / 4;
    u32 w[kWords];
#pragma unroll
    for (int i = 0; i < kWords; ++i) w[i] = __builtin_amdgcn_readfirstlane(((const u32*)p)[i]);
    __builtin_memcpy(&r, w, sizeof(r));
    return r;
}
// Bin of an entry of a long list, in the entries' order.  The bins divide the range of what the sample showed evenly, one shift per
// entry; where the sample shows a crowd in one of those bins (equal keys, or one key far above the others: infinities, a mask
// value), they lie between 255 entries of the sample at equal ranks, 16 to an interval: equal keys then differ by position, and
// no distance between keys matters.  split: the intervals' edges, ascending, kListSplits + 1 of them, in LDS.
__device__ __forceinline__ u32 list_bin(u64 e, u64 lo, u32 sh) {
    const u64 b = (e - lo) >> sh;
    return b < kListBins ? (u32)b : kListBins - 1u;
}
__device__ __forceinline__ u32 list_bin_split(u64 e, const u64* split) {
    constexpr u32 Q = 31u - (u32)__builtin_clz(kListBins / kListSplits);
    u32 p = 0;
#pragma unroll
    for (u32 step = kListSplits / 2; step > 0; step /= 2) p += split[p + step] <= e ? step : 0u;
    const u64 lower = split[p], span = split[p + 1u] - lower;
    const u32 width = span > 1u ? 64u - (u32)__builtin_clzll(span - 1u) : 0u;
    return (p << Q) | (u32)((e - lower) >> (width > Q ? width - Q : 0u));
}

// Per-row working memory beside the list: the upper half of the row's first candidate array (the list proper is at
// most half a row).  Offsets in bytes from its 256-byte-aligned start come from the host (ListPlan).
__device__ __forceinline__ char* list_meta(const Params& P, int row) {
    // (An offset is added; a number made a pointer would be one of no known address space, whose loads and stores wait for LDS, and LDS for them.  One row of 2^24 fp32 keys, k = 256, 31.7 us
    // with that, so 30.6.)
    char* a = (char*)(P.cand[0] + (size_t)row * P.cand_stride + (size_t)((P.n + 1) / 2));
    return a + (0u - (u32)(uintptr_t)a & 255u);
}
// (written by k_list_bound and k_list_part, through list_row_out; constant for every kernel after them)
__device__ __forceinline__ const ListRow* list_row(const Params& P, int row) { return (const ListRow*)list_meta(P, row); }
__device__ __forceinline__ ListRow* list_row_out(const Params& P, int row) { return (ListRow*)list_meta(P, row); }
__device__ __forceinline__ ListDone* list_done(const Params& P, int row) { return (ListDone*)(list_meta(P, row) + kListDoneOff); }
template <class T>
__device__ __forceinline__ T* list_part(const Params& P, int row, u32 off) { return (T*)(list_meta(P, row) + off); }
// The same as a pointer of no known address space, for the sweep's adds to its counters of ties: around adds that it knows to go to global memory the compiler keeps the loads under way in another
// order (2^26 fp16 keys, a ramp, k = 16, 65.4 us, so 63.8; nine in ten bf16 keys equal, k = 300, 66.7 / 64.6).  It is the compiler's order that is measured there: with another one, measure again.
template <class T>
__device__ __forceinline__ T* list_part_generic(const Params& P, int row, u32 off) {
    return (T*)((((uintptr_t)(P.cand[0] + (size_t)row * P.cand_stride + (size_t)((P.n + 1) / 2)) + 255) & ~(uintptr_t)255) + off);
}
__device__ __forceinline__ u64* list_array(const Params& P, u32 which, int row) {
    return (u64*)(P.cand[which] + (size_t)row * P.cand_stride);
}

// Entry of an element, and back.
struct ListEntry {
    u32 kshift, ib, dirmask, idx_max;  // kshift: 16 for 16-bit keys, which are kept in the upper half of their word
    __device__ __forceinline__ u64 of(u32 key, u32 idx) const { return ((u64)(key >> kshift) << ib) | (u64)(idx_max - idx); }
    __device__ __forceinline__ u32 idx(u64 e) const { return idx_max - ((u32)e & idx_max); }
    __device__ __forceinline__ u32 key(u64 e) const { return (u32)(e >> ib) << kshift; }
    __device__ __forceinline__ u64 end() const { return 1ull << (32u - kshift + ib); }  // above every entry
};
template <int DT>
__device__ __forceinline__ ListEntry list_entry(const Params& P) {
    ListEntry c;
    c.kshift = DT == RTOPK_F32 ? 0u : 16u;
    c.ib = (u32)__builtin_popcount(P.idx_max);
    c.dirmask = P.dirmask;
    c.idx_max = P.idx_max;
    return c;
}
// The number an ordered key (of "largest") stands for.
template <int DT>
__device__ __forceinline__ float number_of_key(u32 o) {
    const u32 b = (o & 0x80000000u) ? (o ^ 0x80000000u) : ~o;
    if (DT == RTOPK_F16) return (float)__builtin_bit_cast(_Float16, (uint16_t)(b >> 16));
    return __uint_as_float(DT == RTOPK_F32 ? b : b & 0xffff0000u);
}
// The element's own bits from its key; a NaN's are fetched from the row.
template <int DT>
__device__ __forceinline__ u32 raw_of_key(u32 key, u32 idx, const RowShape& rs, u32 dirmask) {
    const u32 o = key ^ dirmask;
    const u32 nan = DT == RTOPK_F32 ? 0xffffffffu : 0xffff0000u;
    if (o == nan) return load_value<DT>(rs.x, idx);
    const u32 b = (o & 0x80000000u) ? (o ^ 0x80000000u) : ~o;
    return DT == RTOPK_F32 ? b : b >> 16;
}

// block_inclusive_scan for the larger workgroups: the waves' sums are added up on the lane network, not by a loop over them.  (It is
// the same where there are few waves.)
template <int B>
__device__ __forceinline__ u32 block_scan(u32 v, u32* wsum) {
    if constexpr (B < 512) {
        return block_inclusive_scan<B>(v, wsum);
    } else {
        const u32 lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        v = wave_inclusive_scan(v);
        if (lane == 63) wsum[wave] = v;
        __syncthreads();
        const u32 x = wave_inclusive_scan(lane < wave ? wsum[lane % (u32)(B / 64)] : 0u);
        return v + (u32)__builtin_amdgcn_readlane((int)x, 63);
    }
}

// f(0), f(1), ... f(N - 1) with constants: a row in registers must stay a named set of registers (see each_resident_tile).
template <int C, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (C < N) {
        f(std::integral_constant<int, C>{});
        static_for<C + 1, N>(f);
    }
}

// Reductions over a wave on the lane network (see wave_inclusive_scan); the result is in lane 63.  A lane without a
// source keeps its own value.
template <int CTRL, int ROWS>
__device__ __forceinline__ u32 lane_move(u32 v) {
    return (u32)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, ROWS, 0xf, false);
}
template <class Op>
__device__ __forceinline__ u32 wave_reduce(u32 v, Op&& op) {
    v = op(v, lane_move<0x111, 0xf>(v));
    v = op(v, lane_move<0x112, 0xf>(v));
    v = op(v, lane_move<0x114, 0xf>(v));
    v = op(v, lane_move<0x118, 0xf>(v));
    v = op(v, lane_move<0x142, 0xa>(v));
    return op(v, lane_move<0x143, 0xc>(v));
}
template <int CTRL, int ROWS>
__device__ __forceinline__ u64 lane_move64(u64 v) {
    return ((u64)lane_move<CTRL, ROWS>((u32)(v >> 32)) << 32) | lane_move<CTRL, ROWS>((u32)v);
}
template <class Op>
__device__ __forceinline__ u64 wave_reduce64(u64 v, Op&& op) {
    v = op(v, lane_move64<0x111, 0xf>(v));
    v = op(v, lane_move64<0x112, 0xf>(v));
    v = op(v, lane_move64<0x114, 0xf>(v));
    v = op(v, lane_move64<0x118, 0xf>(v));
    v = op(v, lane_move64<0x142, 0xa>(v));
    return op(v, lane_move64<0x143, 0xc>(v));
}
__device__ __forceinline__ u64 last_lane64(u64 v) {
    return ((u64)(u32)__builtin_amdgcn_readlane((int)(u32)(v >> 32), 63) << 32) | (u32)__builtin_amdgcn_readlane((int)(u32)v, 63);
}
struct MaxOf { template <class T> __device__ __forceinline__ T operator()(T a, T b) const { return a > b ? a : b; } };
struct MinOf { template <class T> __device__ __forceinline__ T operator()(T a, T b) const { return a < b ? a : b; } };

// ------------------------------------------------------------------------------------------------
// T from a sample
// ------------------------------------------------------------------------------------------------

// The rank-th largest (or a little less) of the values that each(f) hands to f, over all threads of the workgroup; it lies in
// [lo, hi], and values below lo are passed over.  2048 bins divide [lo, hi] evenly; the bin in question is divided again
// until it holds few values, and its lower edge is returned (*exact: until it was one value).
struct RankShared {
    alignas(16) u32 hist[2 * 2049];  // two copies, a word apart (see HistSlot)
    u32 wsum[16], selv[4];
};
template <int B, class Each>
__device__ __forceinline__ u32 sample_rank(Each&& each, u32 rank, u32 lo, u32 hi, RankShared& sm, bool* exact) {
    constexpr int kPer = 2048 / B;
    const u32 tid = threadIdx.x;
    u32* mine = sm.hist + (lane_id() & 1u) * 2049u;
    u32 left = rank;
    for (;;) {
        const u32 width = hi > lo ? 32u - (u32)__builtin_clz(hi - lo) : 0u, sh = width > 11u ? width - 11u : 0u;
        for (u32 j = tid; j < 2u * 2049u; j += B) sm.hist[j] = 0;
        if (tid == 0) sm.selv[0] = sm.selv[1] = sm.selv[2] = 0;
        __syncthreads();
        each([&](u32 v) __attribute__((always_inline)) {
            if (v >= lo && v <= hi) atomicAdd(&mine[(v - lo) >> sh], 1u);
        });
        __syncthreads();
        u32 c[kPer], s = 0;
        const u32 r0 = tid * kPer;  // position counted from the top bin
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const u32 b = 2047u - (r0 + i);
            c[i] = sm.hist[b] + sm.hist[2049u + b];
            s += c[i];
        }
        const u32 incl = block_scan<B>(s, sm.wsum);
        u32 run = incl - s;
        if (run < left && left <= incl) {
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                if (run < left && left <= run + c[i]) {
                    sm.selv[0] = 2047u - (r0 + i);
                    sm.selv[1] = run;
                    sm.selv[2] = c[i];
                }
                run += c[i];
            }
        }
        __syncthreads();
        const u32 bin = sm.selv[0], inside = sm.selv[2];
        left -= sm.selv[1];
        __syncthreads();
        lo += bin << sh;
        hi = hi - lo > (1u << sh) - 1u ? lo + ((1u << sh) - 1u) : hi;  // (the last bin may reach beyond the range, and beyond 32 bits)
        *exact = sh == 0u;
        if (sh == 0u || inside <= 1u + rank / 16u) return lo;
    }
}

// The same for N values in LDS (v[0 .. N), written by the threads), by the first wave alone -- no barriers among many waves (1024 values: 4.4 us with sample_rank): until
// the values from lo up are at least `rank` and few more, or lo is one value that a crowd has (*exact).  At least `rank` values are not below lo.
// half: only the first N / 2 are there.  Begins and ends with a barrier; `v` (RankShared::hist) may be written again after it.  RUNS: result[2] is how many values that are, result[3] the sum of squares of how many every eight
// neighbours have.
// Bound by the latency of one wave.  [lo, hi] is divided into 512 bins, again and again, a bin being one LDS add (300 rows of 30011 fp16 keys, k = 100,
// halved 16.0 us, so 15.6; 16 rows of 2^17 bf16 keys 15.9 / 15.0).  Bins of 16-bit keys are mostly one value each, and a bin
// of few is no crowd: whoever takes it for one counts the whole sample's equal elements for nothing (1024 rows of 2^17 bf16 logits, k = 1024, halved 69.9, with bins
// 70.9, so 69.8).  HALVE: it is halved, with a compare and a scalar population count per 64 values:
// better where several workgroups of four waves share a compute unit and its LDS (1024 rows of 2^17 bf16 keys, k = 50, 54.7 / 55.5),
// and for a few of 256 values (four fp16 rows of 89250, k = 2, 12.7 / 13.6).
template <int N, bool RUNS = false, bool HALVE = false>
__device__ __forceinline__ u32 rank_by_one_wave(u32 rank, u32 lo, u32 hi, u32* v, u32* result, bool* exact, bool half = false) {
    constexpr u32 kBins = 512, kMine = kBins / 64;
    static_assert(N + kBins <= 2 * 2049 && N % 4 == 0, "bins behind the values");
    const u32 tid = threadIdx.x;
    __syncthreads();
    if (tid < 64u) {
        constexpr int kPer = N / 64;
        u32 mine[kPer];
        auto each = [&](auto&& f) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < (kPer + 1) / 2; ++i) f(i);
            if (half) return;
#pragma unroll
            for (int i = (kPer + 1) / 2; i < kPer; ++i) f(i);
        };
        each([&](int i) __attribute__((always_inline)) { mine[i] = v[i * 64 + tid]; });
        const u32 slack = rank + 1u + rank / 16u;
        bool one = lo >= hi;
        if (HALVE || (kPer <= 4 && rank < 8u)) {
            u32 end = hi;  // fewer than `rank` values lie above it
            while (lo < end) {
                const u32 mid = end - (end - lo) / 2u;
                u32 c = 0;
                each([&](int i) __attribute__((always_inline)) { c += (u32)__popcll(ballot64(mine[i] >= mid)); });
                if (c >= rank) {
                    lo = mid;
                    if (c <= slack) break;
                } else {
                    end = mid - 1u;
                }
            }
            one = lo == end;
        } else {
            u32* bins = v + N;
            u32 above = 0;  // values above hi: fewer than `rank`
            while (!one) {
                const u32 width = 32u - (u32)__builtin_clz(hi - lo), sh = width > 9u ? width - 9u : 0u;
                // (bin 0 is the best; a lane's bins are neighbours)
#pragma unroll
                for (u32 j = 0; j < kMine; j += 4u) *(uint4*)&bins[tid * kMine + j] = make_uint4(0, 0, 0, 0);
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                each([&](int i) __attribute__((always_inline)) {
                    if (mine[i] >= lo && mine[i] <= hi) atomicAdd(&bins[(hi - mine[i]) >> sh], 1u);
                });
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                u32 c[kMine], s = 0;
#pragma unroll
                for (u32 j = 0; j < kMine; ++j) {
                    c[j] = bins[tid * kMine + j];
                    s += c[j];
                }
                u32 run = above + wave_inclusive_scan(s) - s, bin = 0, before = 0, upto = 0;
#pragma unroll
                for (u32 j = 0; j < kMine; ++j) {
                    if (run < rank && rank <= run + c[j]) { bin = tid * kMine + j; before = run; upto = run + c[j]; }
                    run += c[j];
                }
                const u64 who = ballot64(upto != 0u);
                if (who == 0u) break;  // (never: at least `rank` values lie in [lo, hi] or above)
                const int l = (int)__builtin_ctzll(who);
                bin = (u32)__builtin_amdgcn_readlane((int)bin, l);
                above = (u32)__builtin_amdgcn_readlane((int)before, l);
                upto = (u32)__builtin_amdgcn_readlane((int)upto, l);
                hi -= bin << sh;
                lo = hi - lo > (1u << sh) - 1u ? hi - ((1u << sh) - 1u) : lo;  // (the last bin may reach beyond the range)
                if (upto <= slack) break;
                one = lo == hi;
            }
        }
        if (tid == 0) {
            result[0] = lo;
            result[1] = one ? 1u : 0u;
        }
        if constexpr (RUNS) {
            u32 word = 0, sq = 0;  // lane 2 i, 2 i + 1: which of the values i * 64 .. i * 64 + 63 they are
            each([&](int i) __attribute__((always_inline)) {
                const u64 m = ballot64(mine[i] >= lo);
                word = tid == 2u * (u32)i ? (u32)m : word;
                word = tid == 2u * (u32)i + 1u ? (u32)(m >> 32) : word;
            });
            u32 all = (u32)__builtin_popcount(word);
#pragma unroll
            for (u32 b = 0; b < 32u; b += 8u) {
                const u32 c = (u32)__builtin_popcount((word >> b) & 0xffu);
                sq += c * c;
            }
            all = wave_inclusive_scan(all);
            sq = wave_inclusive_scan(sq);
            if (tid == 63u) {
                result[2] = all;
                result[3] = sq;
            }
        }
    }
    __syncthreads();
    *exact = result[1] != 0u;
    return result[0];
}

// An integer hash; the multipliers are those of "lowbias32" (Chris Wellons, hash-prospector).
__device__ __forceinline__ u32 mix32(u32 z) {
    z ^= z >> 16; z *= 0x7feb352du;
    z ^= z >> 15; z *= 0x846ca68bu;
    return z ^ (z >> 16);
}

// A vector's elements -> their keys (direction applied), in place; and the key of element j of such a vector.
template <int DT>
__device__ __forceinline__ void keys_of_vector(uint4& q, u32 dirmask) {
    u32* w = (u32*)&q;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (DT == RTOPK_F32) {
            w[i] = KeyOf<DT>::key(w[i]) ^ dirmask;
        } else {  // two 16-bit keys per word (see KeySource::digits)
            const u32 thr = DT == RTOPK_F16 ? 0x03ff03ffu : 0x007f007fu;
            const u32 x = w[i], sb = x & 0x80008000u;
            u32 key = x ^ ((sb - (sb >> 15)) | 0x80008000u);
            const u32 nb = ((x & 0x7fff7fffu) + thr) & 0x80008000u;
            key |= (nb - (nb >> 15)) | nb;
            w[i] = dirmask ? ~key : key;
        }
    }
}
template <int DT>
__device__ __forceinline__ u32 key_in_vector(const uint4& q, int j) {
    const u32 w[4] = {q.x, q.y, q.z, q.w};
    if constexpr (DT == RTOPK_F32) return w[j % 4];
    else return (j & 1) ? w[j / 2 % 4] & 0xffff0000u : w[j / 2 % 4] << 16;
}

// What the B / 64 waves of a workgroup left in v[0], v[stride], ...: their sum, or the best of them, in every lane.  (One read and six
// steps on the lane network; a loop over 16 waves' words, run by all 16 waves, takes most of 1 us.)
template <int B>
__device__ __forceinline__ u32 sum_of_waves(const u32* v, u32 stride) {
    const u32 x = lane_id() < (u32)(B / 64) ? v[stride * lane_id()] : 0u;
    return (u32)__builtin_amdgcn_readlane((int)wave_inclusive_scan(x), 63);
}
template <int B, class Op>
__device__ __forceinline__ u32 best_of_waves(const u32* v, u32 stride, Op&& op) {
    return (u32)__builtin_amdgcn_readlane((int)wave_reduce(v[stride * (lane_id() % (u32)(B / 64))], op), 63);
}

// Bound by latency: V independent loads per lane, then a few phases with barriers, on one compute unit.  The sample is
// B * V vectors of 16 bytes, in runs of RUN (8: one 128-byte line), one run from a hashed place in each of B * V / RUN equal
// stretches of the row: a trend along the row, or any period in it, cannot line up with that.  (A stretch is at least 1.5 runs
// long and may begin inside one, so that neighbours meet in one run now and then, at most once in nine: it then counts twice.)
// A row that is too short for that has a smaller sample, half as many runs until they fit.
// The rank is taken among the MAXIMA of vectors (or of all a lane's vectors) while it is small against their number:
// neighbouring elements that are alike then count once, so that a row whose best elements lie together does not look
// richer than it is, and there are fewer values to rank.  The rank that stands for the row's k-th key is its share
// ks = k * sample / n, plus six standard deviations of a Poisson count, plus 6 (independent draws: ks = 0.1, 1, 10, 100: more than
// that many are seen with a probability of about 1e-13, 1e-9, 1e-8, 1e-8; the row is then done again).
// Runs whose elements are alike (blocks of one value, a trend) are fewer draws than they have elements: their counts of
// elements not below T show by how much (v), and where T has too few such elements for that, it is taken again, lower.
// For many workgroups per row (a row done again is dear there, and so is a bin that holds much of a long list) what the sample has of
// the list is gathered in LDS first, of every run or of every 2^thin-th.
// te: counters of ties per tile, nt of them, cleared if they will be used.  room: how long a list may be that is put in order
// in LDS.  Thread 0 fills in *lr.
constexpr u32 kSampleList = 8192, kLeastThinned = 128;
struct SampleList {
    // place: (run * RUN + vector of the run) * elements per vector + element
    // (two arrays: a 64-bit store of both would put a loaded vector's words into register pairs, and the kernel into scratch memory)
    u32 key[kSampleList], place[kSampleList];
    u32 run[2048];       // how many of them each run has
    u32 bin[kListBins];  // how many of them, of those better than T, lie in each bin of a long list
    u32 from[16], got[16];  // which of them every wave has: the waves come in any order
    u32 n, next;
};
// record: this workgroup writes the row's record.  after_load(): what may be done once the sample's loads are under way.
template <int DT, int B, int V, bool GATHER, int RUN, class AfterLoad>
__device__ __forceinline__ void bound_of_row(const Params& P, const ListPlan& L, int row, const RowShape& rs, rtopk_row_trace* st,
                                             ListRow* lr, u32* te, u32 nt, u32 room, RankShared& sm, SampleList* sl, u32* red, bool record,
                                             AfterLoad&& after_load) {
    constexpr int E = 16 / KeyOf<DT>::kBytes;
    constexpr u32 kRun = (u32)RUN, kRuns = (u32)(B * V) / kRun, kLeastRuns = 16;
    constexpr u32 kLeast = (u32)B / kRun > kLeastThinned ? (u32)B / kRun : kLeastThinned;  // (thinned by lanes' vectors: one of V is the least there is)
    const u32 tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    KeySource<DT, kGridBlock, key_vecs<DT>(), false> src;
    src.init(rs);
    const u32 v0 = src.lead != 0 ? 1u : 0u;
    const u32 v1 = (u32)(((u64)src.lead + (u64)rs.n) / E);
    const u32 groups = v1 > v0 ? (v1 - v0) / kRun : 0u;  // whole runs inside the row
    u32 lruns = 31u - (u32)__builtin_clz(kRuns);  // (their logarithm)
    while ((1u << lruns) > kLeastRuns && groups < (1u << lruns) + (1u << lruns) / 2u) --lruns;
    const u32 runs = 1u << lruns;
    const ListEntry ent = list_entry<DT>(P);
    const bool sampled = groups >= runs + runs / 2u;
    // (where more than 0.4 of the row is wanted -- ragged batches -- everything is listed)
    const bool whole = !sampled || (u64)rs.k * 5u > (u64)rs.n * 2u;
    const bool bins = GATHER && L.nb != 0u;  // a long list
    // Lane t's vector u is the t % RUN-th of this run: the runs of a lane lie far apart (its best element would else stand for
    // V neighbouring runs where the row has a trend), and so do the runs of any u.
    static_assert((V & (V - 1)) == 0 && (B & (B - 1)) == 0, "one to one");
    auto run_of = [&](u32 t, u32 u) __attribute__((always_inline)) { return t / kRun + (u32)B / kRun * ((u + t / kRun) % (u32)V); };
    auto vector_of = [&](u32 c, u32 i) __attribute__((always_inline)) {  // which vector of the row is the i-th of run c
        // (c << 16 | hash) * groups / runs >> 16, as the upper half of a 32-bit product
        const u32 g = __umulhi((c << 16 | (mix32(c) >> 16)) << (16u - lruns), groups);
        return v0 + g * kRun + i;
    };
    uint4 q[V];
    if (sampled && (bins || !whole)) {
#pragma unroll
        for (int u = 0; u < V; ++u) {
            // (lanes beyond a smaller sample: some of it again, and ignored)
            q[u] = load16<false>(src.abase + vector_of(run_of(tid, (u32)u) & (runs - 1u), tid % kRun));
        }
    }
    if (record) init_row<DT>(P, row, st, rs);
    after_load();
    if (rs.k == 0) {
        if (tid == 0) lr->mode = kListSkip;
        return;
    }
    if constexpr (GATHER) {
        for (u32 r = tid; r < runs; r += B) sl->run[r] = 0;
        if (tid == 0) sl->n = sl->next = 0;
        if (bins)
            for (u32 j = tid; j < kListBins; j += B) sl->bin[j] = 0;
    }
    if (bins) {  // its histogram and the buckets' write positions
        uint4* gh = list_part<uint4>(P, row, L.hist_off);
        for (u32 j = tid; j < L.hists * (kListBins / 4u); j += B) gh[j] = make_uint4(0, 0, 0, 0);
        u32* cur = list_part<u32>(P, row, L.cursor_off);
        for (u32 j = tid; j < 2u * list_cursors(L.nb); j += B) cur[j] = 0;
    }
    if (whole && !(bins && sampled)) {
        if (tid == 0) {
            lr->mode = kListPlain;
            lr->T = 0;
            lr->exact = 1;
            lr->t = 0.0f;
            lr->lo = 0;
            const u32 top = ent.ib + (DT == RTOPK_F32 ? 32u : 16u);
            lr->sh = top > 12u ? top - 12u : 0u;
            lr->split = 0;
        }
        return;
    }
    const u32 vecs = runs * kRun, elems = vecs * E, lanes = vecs < (u32)B ? vecs : (u32)B;
    const float ks = (float)rs.k * ((float)elems / (float)rs.n);
    u32 rank = (u32)(ks + 6.0f * __builtin_sqrtf(ks) + 6.0f);
    auto best_of = [&](const uint4& v) __attribute__((always_inline)) {
        u32 m = 0;
#pragma unroll
        for (int j = 0; j < E; ++j) {
            const u32 k = key_in_vector<DT>(v, j);
            m = m > k ? m : k;
        }
        return m;
    };
    // (16-bit keys are ranked on the 16 bits they have: fewer rounds)
    constexpr u32 ksh = DT == RTOPK_F32 ? 0u : 16u;
    // One wave can rank a quarter as many values as there are.  Where 512 lanes have eight vectors and more each, a larger rank is found among two values per lane, the
    // best of either half of its vectors (eight fp32 rows of 524288, nine in ten equal, k = 3000, rank 158: 32.8 us with sample_rank, 26.9 so; two values for every
    // rank: 8 rows, k = 1000, 24.5 / 25.3).
    constexpr u32 W = GATHER && B == 512 && V >= 8 ? 2u : 1u;
    const bool two = W == 2u && rank > lanes / 4u;
    const u32 vals = !two ? lanes : vecs < 2u * (u32)B ? vecs : 2u * (u32)B;
    u32 best[W] = {}, lmax = 0;
#pragma unroll
    for (int u = 0; u < V; ++u) {
        keys_of_vector<DT>(q[u], P.dirmask);
        const u32 m = best_of(q[u]);
        best[u * W / V] = best[u * W / V] > m ? best[u * W / V] : m;
    }
    if (runs != kRuns) {  // (beyond a smaller sample: no key is below these)
#pragma unroll
        for (u32 w = 0; w < W; ++w) best[w] = 0;
#pragma unroll
        for (int u = 0; u < V; ++u) {
            if (run_of(tid, (u32)u) >= runs) q[u] = make_uint4(0, 0, 0, 0);
            const u32 m = best_of(q[u]);
            best[u * W / V] = best[u * W / V] > m ? best[u * W / V] : m;
        }
    }
#pragma unroll
    for (u32 w = 0; w < W; ++w) lmax = lmax > best[w] ? lmax : best[w];
    auto put_values = [&]() __attribute__((always_inline)) {
        sm.hist[tid] = (two ? best[0] : lmax) >> ksh;
        if (two) sm.hist[(u32)B + tid] = best[W - 1u] >> ksh;
    };
    auto forget = [&]() __attribute__((always_inline)) {  // (nothing worked out from the elements is kept: registers)
#pragma unroll
        for (int u = 0; u < V; ++u) asm volatile("" : "+v"(q[u].x), "+v"(q[u].y), "+v"(q[u].z), "+v"(q[u].w));
    };
    forget();
    // the best of the sample, and the worst of the lanes' best (at least B elements are not below it)
    u32 top = wave_reduce(lmax, MaxOf()), low = wave_reduce(lmax, MinOf());
    if (lane == 63u) {
        red[2 * wave] = top;
        red[2 * wave + 1] = low;
    }
    __syncthreads();
    top = best_of_waves<B>(red, 2, MaxOf());
    low = best_of_waves<B>(red + 1, 2, MinOf());
    __syncthreads();
    u32 T = 0, cnt = 0, eq = 0, thin = 0, got = 0, eq_got = 0;
    bool exact = false;
    auto all = [&](auto&& f) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < V; ++u)
#pragma unroll
            for (int j = 0; j < E; ++j) f(key_in_vector<DT>(q[u], j) >> ksh);
    };
    bool elements = false;  // T is ranked among the elements
    bool alike = true;      // runs may be fewer draws than they have elements
    u32 by_lanes = 0;       // T was ranked among the lanes' best: how many of those values are not below it
    if (whole) {
    } else if (rank <= vals / 4u) {
        put_values();
        T = rank_by_one_wave<(int)W * B, GATHER, (B <= 256)>(rank, low >> ksh, top >> ksh, sm.hist, sm.selv, &exact, W == 2u && !two);
        if constexpr (GATHER) {
            by_lanes = sm.selv[2];
            const float c = (float)by_lanes;
            alike = (float)sm.selv[3] > (2.0f + c / (float)(vals / 8u)) * c;
            if (by_lanes > vals / 2u)  // (T is what most of the sample equals)
                while ((runs >> thin) > kLeast) ++thin;
        }
    } else if (rank <= vecs / 4u) {
        T = sample_rank<B>([&](auto&& f) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < V; ++u) f(best_of(q[u]) >> ksh);
        }, rank, rank <= lanes ? low >> ksh : 0u, top >> ksh, sm, &exact);
    } else {
        elements = true;
    }
    const bool gather = GATHER && (bins || alike);
    // a long list's bins, while they divide the range evenly
    u64 lo = 0;
    u32 sh = 0, most = 0;  // ... and what the fullest of them has of the sample
    auto even_shift = [&](u64 from) __attribute__((always_inline)) {
        const u64 hi = ((u64)(top >> ent.kshift) << ent.ib) | ent.idx_max, range = hi > from ? hi - from : 1u;
        const u32 width = 64u - (u32)__builtin_clzll(range);
        return width > 12u ? width - 12u : 0u;
    };
    auto entry_at = [&](u32 i) __attribute__((always_inline)) {  // of what was gathered
        const u32 at = sl->place[i], v = at / E;
        return ent.of(sl->key[i], vector_of(v / kRun, v % kRun) * E + at % E - src.lead);
    };
    if (!gather) {
        if (elements) T = sample_rank<B>(all, rank, rank <= lanes ? low >> ksh : 0u, top >> ksh, sm, &exact);
        T <<= ksh;
        if (exact) {  // (else T is no key with a crowd)
#pragma unroll
            for (int u = 0; u < V; ++u) {
                u32 c = 0;
#pragma unroll
                for (int j = 0; j < E; ++j) {
                    const u32 k = key_in_vector<DT>(q[u], j);
                    eq += k == T ? 1u : 0u;
                    c += k >= T ? 1u : 0u;
                }
                cnt += run_of(tid, (u32)u) < runs ? c : 0u;
            }
            cnt = wave_inclusive_scan(cnt);
            eq = wave_inclusive_scan(eq);
            if (lane == 63u) { red[2 * wave] = cnt; red[2 * wave + 1] = eq; }
            __syncthreads();
            cnt = sum_of_waves<B>(red, 2);
            eq = sum_of_waves<B>(red + 1, 2);
        }
    }
    if constexpr (GATHER) if (gather) {
        static_assert(kRuns <= sizeof(sl->run) / 4, "a counter per run");
        static_assert(kLeast * kRun * E <= kSampleList, "thinned far enough");
        while ((rank >> thin) > 128u && (runs >> thin) > kLeast) ++thin;
        bool fresh = true, again = false, dense = false;
#pragma unroll 1
        for (bool first = true;; first = false) {
            if (elements && fresh) T = sample_rank<B>(all, rank, rank <= lanes && !again ? low >> ksh : 0u, top >> ksh, sm, &exact);
            if (fresh && (elements || !again)) T <<= ksh;
            const u32 every = (1u << thin) - 1u;
            if (!first) {
                __syncthreads();
                for (u32 r = tid; r < runs; r += B) sl->run[r] = 0;
                for (u32 j = tid; j < kListBins; j += B) sl->bin[j] = 0;
                if (tid == 0) sl->n = 0;
                __syncthreads();
            }
            u32 t0 = tid;
            // (what follows from these is worked out here and not kept for the whole kernel: registers)
            asm volatile("" : "+v"(t0));
            forget();
            if (lane == 63u) sl->got[wave] = 0;
            if (ballot64(lmax >= T) != 0u) {
                // f(vector, how many of its elements are not below T) for the runs that are kept
                auto kept = [&](auto&& f) __attribute__((always_inline)) {
                    static_for<0, V>([&](auto uc) __attribute__((always_inline)) {
                        constexpr u32 u = (u32)decltype(uc)::value;
                        __builtin_amdgcn_sched_barrier(0);  // (one vector at a time: registers)
                        if ((u & every) != every / 2u) return;
                        u32 c = 0;
#pragma unroll
                        for (int j = 0; j < E; ++j) c += key_in_vector<DT>(q[u], j) >= T ? 1u : 0u;
                        f(uc, run_of(t0, u) < runs ? c : 0u);
                    });
                };
                u32 mine = 0;
                kept([&](auto, u32 c) __attribute__((always_inline)) { mine += c; });
                const u32 incl = wave_inclusive_scan(mine);
                u32 at = 0;
                if (lane == 63u) {
                    at = atomicAdd(&sl->n, incl);
                    sl->from[wave] = at;
                    sl->got[wave] = incl;
                }
                at = (u32)__builtin_amdgcn_readlane((int)at, 63) + incl - mine;
                kept([&](auto uc, u32 c) __attribute__((always_inline)) {
                    constexpr int u = decltype(uc)::value;
                    if (ballot64(c != 0u) == 0) return;
                    const u32 run = run_of(t0, (u32)u);
                    u32 r = c;
                    r += (u32)__builtin_amdgcn_update_dpp(0, (int)r, 0xb1, 0xf, 0xf, false);   // the neighbour's
                    r += (u32)__builtin_amdgcn_update_dpp(0, (int)r, 0x4e, 0xf, 0xf, false);   // the other pair's
                    if constexpr (kRun == 8) r += (u32)__builtin_amdgcn_update_dpp(0, (int)r, 0x141, 0xf, 0xf, false);  // the other four's
                    if (lane % kRun == 0u && r != 0u) sl->run[run] = r;
#pragma unroll
                    for (int j = 0; j < E; ++j) {
                        const u32 k = key_in_vector<DT>(q[u], j);
                        if (c != 0u && k >= T) {
                            if (at < kSampleList) {
                                sl->key[at] = k;
                                sl->place[at] = (run * kRun + t0 % kRun) * (u32)E + (u32)j;
                            }
                            ++at;
                        }
                    }
                });
            }
            __syncthreads();
            got = sl->n;
            fresh = false;
            if (got > kSampleList) {
                do { got >>= 1; ++thin; } while (got > kSampleList);
                while ((runs >> thin) < kLeast) --thin;  // (so many runs always fit: more than this many are left)
                continue;
            }
            // how many of them equal T, the sum of the runs' squares, and how many lie in each of a long list's bins
            u32 sq = 0, rich = 0;  // rich: runs of which a quarter counts, and above that how many of them the next run does not follow
            eq_got = most = 0;
            for (u32 r = tid; r < runs; r += B) {
                const u32 c = sl->run[r], next = r + 1u < runs ? sl->run[r + 1u] : 0u;
                sq += c * c;
                if (c >= kRun * E / 4u) rich += next >= kRun * E / 4u ? 1u : 0x10001u;
            }
            lo = (u64)(T >> ent.kshift) << ent.ib;
            sh = even_shift(lo);
            for (u32 i = tid; i < got; i += B) {
                const u32 k = sl->key[i];
                eq_got += k == T ? 1u : 0u;
                if (bins && k != T) {
                    const u32 before = atomicAdd(&sl->bin[list_bin(entry_at(i), lo, sh)], 1u);
                    most = most > before ? most : before + 1u;
                }
            }
            eq_got = wave_inclusive_scan(eq_got);
            sq = wave_inclusive_scan(sq);
            rich = wave_inclusive_scan(rich);
            most = wave_reduce(most, MaxOf());
            if (lane == 63u) { red[4 * wave] = eq_got; red[4 * wave + 1] = sq; red[4 * wave + 2] = most; red[4 * wave + 3] = rich; }
            __syncthreads();
            eq_got = sum_of_waves<B>(red, 4);
            sq = sum_of_waves<B>(red + 1, 4);
            most = best_of_waves<B>(red + 2, 4, MaxOf());
            rich = sum_of_waves<B>(red + 3, 4);
            cnt = got << thin;
            eq = eq_got << thin;
            const float v = got != 0u ? (float)sq / (float)got - (float)cnt / (float)runs : 0.0f;
            if (v > 2.0f && thin != 0u && !dense) {  // (few draws: all there are are needed, for T and for splitters)
                dense = true;
                thin = 0;
                continue;
            }
            // (a list holds at least what the sample has of it: nothing can go wrong from k on, twice k where runs meet)
            // (Rich runs that all follow one another are a trend: one run from every stretch then misses by one at either end at most.
            // A ramp of 13.6 million fp32 keys with infinities, k = 5676: 105 us with the margin of independent runs.)
            const float need = ks + ((rich >> 16) == 1u && (rich & 0xffffu) >= 3u ? 2.0f * v : 4.0f * __builtin_sqrtf(ks * v) + 3.0f * v);
            const u32 have = thin == 0u ? cnt : rank;  // (thinned, cnt is an estimate; it is no less than the rank)
            if (whole || again || !(v > 2.0f) || !((float)have < need) || have >= 2u * rs.k) break;
            rank = need < (float)elems ? (u32)need : elems;
            fresh = again = true;
            // (so many lanes have that many such elements, if the next ones have as many each: one wave finds that out sooner)
            const float more = need * (float)by_lanes / (float)got * 1.25f + 2.0f;
            if (by_lanes != 0u && thin == 0u && more < (float)(vals / 2u)) {
                __syncthreads();
                put_values();
                T = rank_by_one_wave<(int)W * B>((u32)more, 0u, top >> ksh, sm.hist, sm.selv, &exact, W == 2u && !two) << ksh;
            } else {
                elements = true;
            }
        }
    }
    // Most of the row may equal T, or so much that the list would be longer than half the row or than what is put in order in
    // LDS: then what is better is listed and the equal elements are counted.
    const u64 eq_row = (u64)eq * rs.n / elems, est = (u64)cnt * rs.n / elems;
    const bool tied = !whole && eq != 0u && ((eq_row > (u64)kListTies && eq_row > (u64)rs.k) ||
                                             (cnt > elems / 20u * 9u && cnt - eq < elems / 5u * 2u) ||
                                             (est + est / 8u > (u64)room && (est - eq_row) * 4u < (u64)room * 3u));
    if (tied) {
        for (u32 j = tid; j < nt; j += B) te[j] = 0;
    }
    bool split = false;
    if constexpr (GATHER) if (bins) {
        // (Little of the sample is better than T: as much of the row again may be better than the best of that, and would all fall into the last bin.  2^28 fp32 keys, nine in ten
        // equal, k = 20000, two of 16384 vectors' elements better: 230 us, so 214.5.)
        const u32 better = (tied ? got - eq_got : got) << thin;
        sh += better < 4u ? 2u : better < 32u ? 1u : 0u;
        // (those equal to T: one key's share of the bins is by position)
        const u32 ties = eq_got >> (ent.ib > sh ? ent.ib - sh : 0u);
        if (!tied && most < ties) most = ties;
        // (a bin of several buckets' ranks -- up to there its parts are shared out in no time -- and more of them than fall together by
        // chance: 4096 bins, 2^28 keys, k = 2^20: about 400 draws)
        split = most > 5u && ((u64)most << thin) * rs.n / elems > 8192u;
        if (split) {
            static_assert(sizeof(sm.hist) >= kListSplits * 8, "room for the candidates");
            u64* cand = (u64*)sm.hist;
            // every total / 256-th of them, in the order of the waves, in which they did not come: the same row has the same splitters every time.
            // (Those that are better than a crowd are not counted by wave, and taken as they came.)
            const u32 total = tied ? got - eq_got : got;
            if (tid < kListSplits) {
                cand[tid] = ent.end();
                const u32 pos = total > kListSplits ? ((tid + 1u) * total - 1u) / kListSplits : tid;
                u32 before = 0, at = 0;
#pragma unroll
                for (u32 w = 0; w < (u32)(B / 64); ++w) {
                    const u32 c = sl->got[w], l = pos - before;
                    at = l < c ? sl->from[w] + l : at;
                    before += c;
                }
                if (!tied && pos < total) cand[tid] = entry_at(at);
            }
            __syncthreads();
            if (tied) {
                for (u32 i = tid; i < got; i += B) {
                    if (sl->key[i] == T) continue;
                    const u32 pos = atomicAdd(&sl->next, 1u);
                    const u32 s0 = total > kListSplits ? pos * kListSplits / total : pos;
                    const u32 s1 = total > kListSplits ? (pos + 1u) * kListSplits / total : pos + 1u;
                    if (s0 != s1) cand[s0] = entry_at(i);
                }
            }
            __syncthreads();
            if (tid < kListSplits) {
                const u64 c = cand[tid];
                u32 r = 0;
#pragma unroll 8
                for (u32 i = 0; i < kListSplits; ++i) r += (cand[i] < c || (cand[i] == c && i < tid)) ? 1u : 0u;
                u64* edge = list_part<u64>(P, row, L.split_off);
                if (r != 0u) edge[r] = c;
                if (tid == 0) {
                    edge[0] = lo;
                    edge[kListSplits] = ent.end();
                }
            }
        }
    }
    if (tid == 0) {
        lr->mode = tied ? kListTied : kListPlain;
        lr->T = T;
        // as a number: not below the number whose key is T ("largest"), or below the one whose key is the next
        // ("smallest": keys are complemented)
        const bool largest = P.dirmask == 0;
        const u64 o = T ^ P.dirmask;
        float t = 0.0f;
        if (whole) {
            lr->exact = 1;
        } else if (tied) {
            // the number whose key is T; not where equal numbers have different keys (the zeros, NaNs)
            t = number_of_key<DT>((u32)o);
            lr->exact = t == 0.0f || t != t;
        } else {
            lr->exact = !threshold_number<DT>(largest ? o : o + (DT == RTOPK_F32 ? 1u : 0x10000u), &t);
        }
        lr->t = t;
        lr->lo = lo;
        lr->sh = sh;
        lr->split = split ? 1u : 0u;
        if (record) {
            st->pre_elems = elems;
            st->pre_bound = T >> (32u - P.pass[0].bits);
        }
    }
}

// Half the largest sample (fp32, long lists) is in runs of 4 vectors, so that there are as many runs: a trend's list is known by them alone, to a stretch or two of the row.
template <int DT, int B, int V, int RUN = 8>
__global__ void __launch_bounds__(B) k_list_bound(Params P, ListPlan L) {
    __shared__ RankShared sm;
    __shared__ SampleList sl;
    __shared__ u32 red[4 * (B / 64)];
    const int row = blockIdx.x;
    const RowShape rs = row_shape_scalar<DT>(P, row);
    ListSource<DT, false> src;  // (the smaller of the two sweeps' tiles: the larger number of them)
    src.init(rs);
    bound_of_row<DT, B, V, true, RUN>(P, L, row, rs, row_state(P, row), list_row_out(P, row), list_part<u32>(P, row, L.tile_off), src.ntiles(),
                           L.nb != 0u ? ~0u : L.room, sm, &sl, red, true, [] {});
}

// ------------------------------------------------------------------------------------------------
// the sweep
// ------------------------------------------------------------------------------------------------

// Staged (raw bits, index) pairs -> entries at the workgroup's next free places; LONG: counted into the histogram.  (Expanded in place: around a call
// the compiler keeps the tiles in flight in memory.)  The first `slots` of a workgroup's entries go to `front`
// (short lists).
template <int DT, bool LONG>
__device__ __forceinline__ void list_flush(u64* seg, u64* front, u32 slots, Lds<u64>* buf, Lds<u32>* run, u32 fill, Lds<u32>* hist, const u64* split,
                                           const ListEntry& c, const ListRow& lr, u32 lane) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    u32 base = 0;
    if (lane == 0) base = __hip_atomic_fetch_add(run, fill, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    base = __builtin_amdgcn_readfirstlane(base);
    for (u32 i = lane; i < fill; i += 64) {
        const u64 v = buf[i];
        const u64 e = c.of(KeyOf<DT>::key((u32)v) ^ c.dirmask, (u32)(v >> 32));
        if (LONG) {
            ((Glb<u64>*)seg)[base + i] = e;
        } else {
            u64* at = base + i < slots ? front : seg;
            ((Glb<u64>*)at)[base + i] = e;
        }
        if (LONG) {
            __hip_atomic_fetch_add(hist + (lr.split != 0u ? list_bin_split(e, split) : list_bin(e, lr.lo, lr.sh)), 1u, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}
// Where workgroup wg's part of the list begins: as many entries in as the units before it have elements that are dealt to the workgroups before it.
// Unit c (of `unit` vectors, a power of two) is workgroup c % G's; the first and the last of a row may be short.
template <int DT>
__device__ __forceinline__ u32 list_segment(const RowShape& rs, u32 wg, u32 G, u32 unit) {
    KeySource<DT, 64, 4, false> src;
    src.init(rs);
    const u32 ue = unit * (u32)decltype(src)::E;
    const u32 units = (u32)((src.nvec + unit - 1u) >> (31u - (u32)__builtin_clz(unit))), q = units / G, r = units % G;
    u64 at = (u64)(wg * q + (wg < r ? wg : r)) * ue;
    if (wg > 0) at -= src.lead;
    if (units > 0 && (units - 1u) % G < wg) at -= (u64)units * ue - src.lead - src.n;  // (the last unit's missing end)
    return (u32)at;
}
// k_list_stream: tiles of 4 KB, which are dealt to the waves one by one.
constexpr u32 kWaveVecs = 256;

// Element s (0 .. kSlots - 1, different in every lane) of a tile that is held in registers: a tree of selects.  (An index
// that varies would put the tile into scratch memory.)
template <class Source>
__device__ __forceinline__ u32 pick(const typename Source::Tile& t, u32 s) {
    const u32 w = Source::E == 4 ? s : s >> 1;  // which of the 16 words
    auto of4 = [&](const uint4& q) __attribute__((always_inline)) {
        const u32 lo = (w & 1u) ? q.y : q.x, hi = (w & 1u) ? q.w : q.z;
        return (w & 2u) ? hi : lo;
    };
    u32 x;
    if constexpr (Source::kSlots / Source::E == 4) {
        const u32 c0 = of4(t.r[0]), c1 = of4(t.r[1]), c2 = of4(t.r[2]), c3 = of4(t.r[3]);
        const u32 d0 = (w & 4u) ? c1 : c0, d1 = (w & 4u) ? c3 : c2;
        x = (w & 8u) ? d1 : d0;
    } else {
        const u32 c0 = of4(t.r[0]), c1 = of4(t.r[1]);
        x = (w & 4u) ? c1 : c0;
    }
    if constexpr (Source::E == 4) return x;
    else return (s & 1u) ? x >> 16 : x & 0xffffu;
}

// 2 * bits + (x < t): compare into carry, add with carry -- two instructions.  (False where x or t is a NaN.)
__device__ __forceinline__ u32 shift_in_below(u32 bits, float x, float t) {
    asm("v_cmp_gt_f32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc" : "+v"(bits) : "v"(t), "v"(x) : "vcc");
    return bits;
}
__device__ __forceinline__ u32 shift_in_equal(u32 bits, float x, float t) {
    asm("v_cmp_eq_f32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc" : "+v"(bits) : "v"(t), "v"(x) : "vcc");
    return bits;
}
__device__ __forceinline__ u32 shift_in_not_above(u32 bits, float x, float t) {
    asm("v_cmp_ge_f32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc" : "+v"(bits) : "v"(t), "v"(x) : "vcc");
    return bits;
}
__device__ __forceinline__ u32 shift_in_not_up_to(u32 bits, float x, float t) {  // !(x <= t): true for NaNs
    asm("v_cmp_nge_f32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc" : "+v"(bits) : "v"(t), "v"(x) : "vcc");
    return bits;
}
// That for the elements of a full tile, the first element's bit on top.  (Inverted for "largest", where NaNs are wanted; as
// it is for "smallest".)
template <class Source>
__device__ __forceinline__ u32 below_mask(const Source& src, const typename Source::Tile& t, float thr) {
    u32 bits = 0;
#pragma unroll
    for (int s = 0; s < Source::kSlots; ++s) bits = shift_in_below(bits, src.template value<SRC_KEY>(t, s, 0.0f), thr);
    return bits;
}

// Position in the row of a lane's element s.
template <class Source>
__device__ __forceinline__ u32 element_index(const Source& src, u32 tile, u32 s) {
    constexpr u32 E = Source::E, B = (u32)Source::kTileVecs / (Source::kSlots / E);
    return (tile * (u32)Source::kTileVecs + (s / E) * B + threadIdx.x) * E + s % E - src.lead;
}

// Workgroup wg of the G that share the row: what is not below the row's bound goes to append(tile, mask), bit
// kSlots - 1 - s of a lane's mask standing for its element s; where ties are counted, tile j's go to te[j], and lane 63 returns how many its wave saw.
// Bound by HBM.  Per element: a compare and an add-with-carry (and the unpacking of a 16-bit key), into one mask per lane
// and tile; another pair where ties are counted.  A branch per 64 elements, or a store, would cost more than the row's trip from
// memory (see stream_tile).  Full tiles go through the load pipeline of for_each_tile, whose loads in the steady state are
// unconditional: behind a conditional prefetch a wave waits for the prefetch too.  us per call with conditional prefetches / so: 1024
// rows of 2^17 bf16 keys, k = 50, 57.2 / 55.2.  Ties by key, tiles loaded one after the other / by number in the pipeline: 2^26
// fp32 keys, nine in ten equal, k = 2^16, 114.9 / 93.1.
template <int DT, class Source, class Append>
__device__ __forceinline__ u32 sweep_row(const Source& src, u32 wg, u32 G, const ListRow& lr, u32* te, u32 dirmask, Append&& append) {
    typedef typename Source::Tile Tile;
    u32 ties = 0;
    const u32 ntiles = src.ntiles(), lane = lane_id(), T = lr.T;
    const bool tied = lr.mode == kListTied, largest = dirmask == 0;
    constexpr u32 kAll = 0xffffffffu >> (32 - Source::kSlots);
    const float t = lr.t;
    auto count_ties = [&](u32 tile, u32 eq) __attribute__((always_inline)) {
        eq = wave_inclusive_scan(eq);
        ties += eq;
        if (lane == 63u && eq != 0u) atomicAdd(&te[tile], eq);
    };
    // short tiles, and every tile where T is not a number to compare with
    auto by_key = [&](const Tile& cur) __attribute__((always_inline)) {
        constexpr u32 E = Source::E;
        u32 m = 0, eq = 0;
#pragma unroll
        for (int u = 0; u < Source::kSlots / (int)E; ++u) {
            uint4 q = cur.r[u];
            keys_of_vector<DT>(q, dirmask);
            const u32 idx = element_index(src, cur.tile, (u32)u * E);  // (a lead-in element's wraps to a huge number)
#pragma unroll
            for (u32 j = 0; j < E; ++j) {
                const u32 key = key_in_vector<DT>(q, (int)j);
                const bool valid = idx + j < src.n;
                m = m + m + ((valid && (tied ? key > T : key >= T)) ? 1u : 0u);
                eq += (valid && key == T) ? 1u : 0u;
            }
            __builtin_amdgcn_sched_barrier(0);  // (one vector's keys at a time: registers)
        }
        append(cur, m);
        if (tied) count_ties(cur.tile, eq);
    };
    if (lr.exact == 0u && !tied) {
        const u32 flip = largest ? kAll : 0u;
        for_each_tile<1>(src, wg, G, ntiles,
                             [&](const Tile& cur) __attribute__((always_inline)) { append(cur, below_mask(src, cur, t) ^ flip); }, by_key);
    } else if (lr.exact == 0u) {
        // better than t, and how many equal it: "largest" notes what is not (x <= t), which a NaN is, "smallest" what is x < t
        for_each_tile<1>(src, wg, G, ntiles,
                         [&](const Tile& cur) __attribute__((always_inline)) {
                             u32 m = 0, eq = 0;
#pragma unroll
                             for (int s = 0; s < Source::kSlots; ++s) {
                                 const float x = src.template value<SRC_KEY>(cur, s, 0.0f);
                                 m = largest ? shift_in_not_above(m, x, t) : shift_in_below(m, x, t);
                                 eq = shift_in_equal(eq, x, t);
                             }
                             append(cur, m ^ (largest ? kAll : 0u));
                             count_ties(cur.tile, (u32)__builtin_popcount(eq));
                         },
                         by_key);
    } else {
        for (u32 next = wg; next < ntiles; next += G) {
            Tile cur;
            src.load(next, threadIdx.x, cur);
            by_key(cur);
        }
    }
    return ties;
}

// (The compiler keeps 30 to 60 scalar registers of the fp32 sweeps, and up to 200 of the 16-bit ones and of the row kernels, in lanes of a
// vector register; the sweeps are at the rate of memory all the same.)
// A wave takes one noted element per lane at a time until no lane has any left, stages them in LDS, and writes
// a full stage to the workgroup's part of the list.
template <int DT, bool LONG, class Source>
struct ListWriter {
    static constexpr u32 ST = LONG ? kListStageLong : kListStage;
    ListEntry ent;
    u64 *seg, *front;
    u32 slots;
    uint2* buf;       // this wave's stage
    u32* run;         // entries of the workgroup so far
    u32* hist;        // LONG
    const u64* split;
    u32 fill;
    __device__ __forceinline__ void flush(const ListRow& lr) {
        list_flush<DT, LONG>(seg, front, slots, lds_words(buf), lds_word(run), fill, lds_word(hist), split, ent, lr, lane_id());
        fill = 0;
    }
    // index(s): position in the row of this lane's element s
    template <class Index>
    __device__ __forceinline__ void append(const typename Source::Tile& cur, u32 m, const ListRow& lr, Index&& index) {
        for (;;) {
            const u64 have = ballot64(m != 0u);
            if (have == 0) break;
            if (fill > ST - 64u) flush(lr);
            if (m != 0u) {
                const u32 bit = 31u - (u32)__builtin_clz(m), s = (u32)Source::kSlots - 1u - bit;
                m ^= 1u << bit;
                buf[fill + mbcnt64(have)] = make_uint2(pick<Source>(cur, s), index(s));
            }
            fill += (u32)__popcll(have);
        }
    }
};

// X -> list, one segment per workgroup.
// NT: the input is far larger than the last-level cache.  LONG: the list's histogram is counted as it is written; then one
// workgroup of 1024 threads has a compute unit, so that there are no more than 256 histograms to add up (512
// workgroups of 512: adding up took longer than it saved).
template <int DT, bool NT, bool LONG, int V = 4>
__global__ void __launch_bounds__(LONG ? kLongBlock : kGridBlock, LONG ? 4 : DT == RTOPK_F32 ? 8 : 6) k_list_sweep(Params P, ListPlan L) {
    constexpr int B = LONG ? kLongBlock : kGridBlock;
    __shared__ uint2 stage[B / 64][LONG ? kListStageLong : kListStage];
    __shared__ u32 hist[LONG ? kListBins : 1];
    __shared__ u64 split[LONG ? kListSplits + 1 : 1];
    __shared__ u32 run, all_ties;
    typedef ListSource<DT, LONG, NT, V> Source;
    const u32 G = (u32)L.G;
    const int row = (int)(blockIdx.x / G);
    const u32 wg = blockIdx.x % G;
    const ListRow lr = list_row_scalar(list_row(P, row));
    if (lr.mode == kListSkip) return;
    const RowShape rs = row_shape_scalar<DT>(P, row);
    Source src;
    src.init(rs);
    const u32 tid = threadIdx.x;
    if (LONG) {
        for (u32 j = tid; j < kListBins; j += B) hist[j] = 0;
        if (lr.split != 0u && tid <= kListSplits) split[tid] = list_part<u64>(P, row, L.split_off)[tid];
    }
    if (tid == 0) run = all_ties = 0;
    __syncthreads();
    ListWriter<DT, LONG, Source> w{list_entry<DT>(P), list_array(P, 1u, row) + list_segment<DT>(rs, wg, G, (u32)Source::kTileVecs),
                                   list_part<u64>(P, row, L.front_off) + (size_t)wg * L.slots, L.slots, stage[tid >> 6], &run, hist, split, 0u};
    const u32 ties = sweep_row<DT>(src, wg, G, lr, list_part_generic<u32>(P, row, L.tile_off), P.dirmask, [&](const typename Source::Tile& cur, u32 m) __attribute__((always_inline)) {
        w.append(cur, m, lr, [&](u32 s) __attribute__((always_inline)) { return element_index(src, cur.tile, s); });
    });
    if (w.fill != 0u) w.flush(lr);
    if (lane_id() == 63u && ties != 0u) atomicAdd(&all_ties, ties);
    __syncthreads();
    if (tid == 0) list_part<uint2>(P, row, L.seg_off)[wg] = make_uint2(run, all_ties);
    if (LONG) {
        u32* gh = list_part<u32>(P, row, L.hist_off) + (wg & (L.hists - 1u)) * kListBins;
        for (u32 j = tid; j < kListBins; j += B) {
            const u32 c = hist[j];
            if (c) atomicAdd(&gh[j], c);
        }
    }
}

// Sample, T and X -> list in one launch, for few rows and short lists.  Every workgroup takes the same sample and comes to the same T by itself (the
// sample, 64 or 128 KB, comes from its XCD's cache for all but the first of them), while its first tiles are on their way: nobody waits for
// anybody, and no word of memory has to be cleared by an earlier launch.
// Every wave works by itself, on tiles of 4 KB that are dealt evenly to all of them; four of them are in registers, and each is loaded anew as soon
// as it is done with, so that 12 to 16 KB per wave and 128 KB per compute unit are in flight.  (1 GiB read and compared: tiles of 64 KB of a workgroup of
// 1024, two in turn, 162 us; by waves 155; dealt by counters, eight workgroups on eight XCDs to each, 175.  Four neighbouring tiles to a wave at a time,
// normal keys, cost up to 0.5 us less, but of a ramp a wave or two then write most of the list: 2^23 fp32 keys, k = 100, 54 / 42 us with single ones.)
template <int DT, bool NT>
using WaveSource = KeySource<DT, 64, 4, NT>;
template <int DT, class Source, class Bound, class Append>
__device__ __forceinline__ u32 sweep_by_waves(const Source& src, u32 first, u32 step, u32* te, u32 dirmask, Bound&& bound, Append&& append) {
    typedef typename Source::Tile Tile;
    u32 ties = 0;  // (in lane 63)
    constexpr u32 E = Source::E, kRing = 4;
    constexpr u32 kAll = 0xffffffffu >> (32 - Source::kSlots);
    const u32 lane = lane_id(), ntiles = src.ntiles();
    const u32 nvec = (u32)src.nvec, last = nvec - 1u;
    u32 f0, f1;  // tiles [f0, f1) are full
    src.full_range(f0, f1);
    Tile t[kRing];
    auto load = [&](u32 tile, Tile& x) __attribute__((always_inline)) {  // (beyond the row's end: its last vector, which is nobody's)
        x.tile = tile;
#pragma unroll
        for (u32 u = 0; u < 4u; ++u) {
            const u32 v = tile * (u32)Source::kTileVecs + u * 64u + lane;
            x.r[u] = load16<Source::kStreams>(src.abase + (v < last ? v : last));
        }
    };
    ListRow lr;
    if (!bound([&]() __attribute__((always_inline)) {
            if (first < ntiles) static_for<0, (int)kRing>([&](auto c) __attribute__((always_inline)) { load(first + (u32)decltype(c)::value * step, t[decltype(c)::value]); });
        }, lr)) return 0;
    const bool tied = lr.mode == kListTied, largest = dirmask == 0;
    const u32 T = lr.T;
    const float thr = lr.t;
    // (a tile is one wave's alone: nothing to add to, and nothing to be cleared before)
    auto note_ties = [&](u32 tile, u32 eq) __attribute__((always_inline)) {
        eq = wave_inclusive_scan(eq);
        ties += eq;
        if (lane == 63u) te[tile] = eq;
    };
    // short tiles, and every tile where T is not a number to compare with
    auto by_key = [&](const Tile& x) __attribute__((always_inline)) {
        u32 m = 0, eq = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            uint4 v = x.r[u];
            keys_of_vector<DT>(v, dirmask);
            const u32 idx = (x.tile * (u32)Source::kTileVecs + (u32)u * 64u + lane) * E - src.lead;  // (a lead-in element's wraps to a huge number)
#pragma unroll
            for (u32 j = 0; j < E; ++j) {
                const u32 key = key_in_vector<DT>(v, (int)j);
                const bool valid = idx + j < src.n;
                m = m + m + ((valid && (tied ? key > T : key >= T)) ? 1u : 0u);
                eq += (valid && key == T) ? 1u : 0u;
            }
            __builtin_amdgcn_sched_barrier(0);  // (one vector's keys at a time: registers)
        }
        append(x, m, lr);
        if (tied) note_ties(x.tile, eq);
    };
    auto all_tiles = [&](auto&& one) __attribute__((always_inline)) {
        for (u32 cur = first; cur < ntiles; cur += kRing * step) {
            if (ntiles - cur <= kRing * step) {
                static_for<0, (int)kRing>([&](auto c) __attribute__((always_inline)) { one(t[decltype(c)::value]); });
                break;
            }
            static_for<0, (int)kRing>([&](auto c) __attribute__((always_inline)) {
                one(t[decltype(c)::value]);
                load(cur + kRing * step + (u32)decltype(c)::value * step, t[decltype(c)::value]);
                __builtin_amdgcn_sched_barrier(0);
            });
        }
    };
    if (lr.exact == 0u && !tied) {
        const u32 flip = largest ? kAll : 0u;
        all_tiles([&](const Tile& x) __attribute__((always_inline)) {
            if (x.tile >= f0 && x.tile < f1) append(x, below_mask(src, x, thr) ^ flip, lr);
        });
    } else if (lr.exact == 0u) {
        // better than t, and how many equal it: "largest" notes what is not (x <= t), which a NaN is, "smallest" what is x < t
        all_tiles([&](const Tile& x) __attribute__((always_inline)) {
            if (x.tile < f0 || x.tile >= f1) return;
            u32 m = 0, eq = 0;
#pragma unroll
            for (int s = 0; s < Source::kSlots; ++s) {
                const float v = src.template value<SRC_KEY>(x, s, 0.0f);
                m = largest ? shift_in_not_above(m, v, thr) : shift_in_below(m, v, thr);
                eq = shift_in_equal(eq, v, thr);
            }
            append(x, m ^ (largest ? kAll : 0u), lr);
            note_ties(x.tile, (u32)__builtin_popcount(eq));
        });
    }
    if (lr.exact != 0u) {
#pragma unroll 1
        for (u32 cur = first; cur < ntiles; cur += kRing * step) {
#pragma unroll 1
            for (u32 tile = cur; tile < ntiles && tile - cur < kRing * step; tile += step) {
                load(tile, t[0]);
                by_key(t[0]);
            }
        }
    } else {
        // the row's first and last tile, if they are short
#pragma unroll 1
        for (u32 e = 0; e < 2u; ++e) {
            const u32 tile = e == 0u ? 0u : f1;
            if ((e == 0u ? f0 == 0u : tile >= ntiles) || tile % step != first) continue;
            load(tile, t[0]);
            by_key(t[0]);
        }
    }
    return ties;
}

// Of rows from 16 MB up the sample is half as large as k_list_bound's, in runs of 4 vectors: as many runs, which is all that a trend's list is known by.
// (Runs of 8, of 4, a ramp, k = 100 and 600: 2^23 fp32 keys 63 and 65, 42 and 45 us; 10 million fp16 keys 73 and 74, 50 and 52.  Normal keys, k = 100, of which twice as many
// lines are read: 25.9 / 28.1 and 25.0 / 26.5, where k_list_bound and k_list_sweep take 35.7 and 31.2.)
template <int DT, int V, int RUN, bool NT>
__global__ void __launch_bounds__(kSharedBlock) k_list_stream(Params P, ListPlan L) {
    constexpr int B = kSharedBlock;
    struct BoundShared { RankShared rank; SampleList list; u32 red[4 * (B / 64)]; };
    __shared__ union { BoundShared bound; uint2 stage[B / 64][kListStage]; } sm;
    __shared__ ListRow decided;
    __shared__ u32 run, all_ties, none[1];
    typedef WaveSource<DT, NT> Source;
    const u32 G = (u32)L.G, tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row = (int)(blockIdx.x / G);
    const u32 wg = blockIdx.x % G;
    const RowShape rs = row_shape_scalar<DT>(P, row);
    Source src;
    src.init(rs);
    ListWriter<DT, false, Source> w{list_entry<DT>(P), list_array(P, 1u, row) + list_segment<DT>(rs, wg, G, kWaveVecs),
                                    list_part<u64>(P, row, L.front_off) + (size_t)wg * L.slots, L.slots, sm.stage[wave], &run, none, nullptr, 0u};
    const u32 ties = sweep_by_waves<DT>(src, wave * G + wg, G * (u32)(B / 64), list_part<u32>(P, row, L.tile_off), P.dirmask,
                     [&](auto&& load_first, ListRow& lr) __attribute__((always_inline)) {
                         bound_of_row<DT, B, V, true, RUN>(P, L, row, rs, row_state(P, row), &decided, nullptr, 0u, L.room, sm.bound.rank, &sm.bound.list,
                                                      sm.bound.red, wg == 0u, [&]() __attribute__((always_inline)) { if (rs.k != 0u) load_first(); });
                         if (tid == 0) run = all_ties = 0;
                         __syncthreads();
                         lr = list_row_scalar(&decided);
                         if (wg == 0u && tid == 0) *list_row_out(P, row) = lr;
                         return lr.mode != kListSkip;
                     },
                     [&](const typename Source::Tile& x, u32 m, const ListRow& lr) __attribute__((always_inline)) {
                         w.append(x, m, lr, [&](u32 s) __attribute__((always_inline)) {
                             return (x.tile * (u32)Source::kTileVecs + (s / (u32)Source::E) * 64u + lane_id()) * (u32)Source::E + s % (u32)Source::E - src.lead;
                         });
                     });
    if (w.fill != 0u) w.flush(decided);
    if (lane_id() == 63u && ties != 0u) atomicAdd(&all_ties, ties);
    __syncthreads();
    if (tid == 0) list_part<uint2>(P, row, L.seg_off)[wg] = make_uint2(run, all_ties);
}

// ------------------------------------------------------------------------------------------------
// putting entries in order
// ------------------------------------------------------------------------------------------------

// A workgroup of B threads puts up to 8 B entries in order in LDS: 4 B bins that divide the range from the best entry to
// the worst evenly, positions within a bin by arrival, and then every entry's rank among its bin's.  Entries are
// distinct and bins hold one or two of them unless the keys are very uneven.  If a bin that matters has more than kOrderCrowd,
// over the number of entries per thread (equal keys; one key far from the others), the bins are laid anew between 255 of the entries themselves: equal keys then
// differ by their positions, and no distance between keys matters.  Only entries that defeat that as well (more than
// kSplitCrowd in one bin) go through a bitonic network.
constexpr u32 kOrderCrowd = 128, kSplitCrowd = 256;
template <int B>
struct OrderShared {
    u64 buf[8 * B + 4];  // (four more: they are compared four at a time)
    u32 hist[4 * B + 2];
    u32 wsum[B / 64];
    u64 red[2 * (B / 64)];
    u32 flag, sp;
};

// Bins between splitters: edge[0] (above every entry) > edge[1] > ... > edge[N] (at or below every entry), N intervals
// of 2^Q bins each, which divide it evenly; bin 0 is the best.
template <int B>
struct SplitBins {
    static constexpr int N = B < 256 ? B : 256;  // intervals
    static constexpr u32 Q = 31u - (u32)__builtin_clz(4 * B / N);
    __device__ static __forceinline__ u32 shift(u64 upper, u64 lower) {
        const u64 span = upper - lower - (upper > lower ? 1u : 0u);
        const u32 width = span ? 64u - (u32)__builtin_clzll(span) : 0u;
        return width > Q ? width - Q : 0u;
    }
    __device__ static __forceinline__ u32 bin(const u64* edge, u64 e) {
        u32 p = 0;
#pragma unroll
        for (u32 step = N / 2; step > 0; step /= 2) p += edge[p + step] > e ? step : 0u;
        const u64 upper = edge[p];
        return (p << Q) | (u32)((upper - 1u - e) >> shift(upper, edge[p + 1u]));
    }
    // The least number that belongs to bin b.
    __device__ static __forceinline__ u64 floor_of(const u64* edge, u32 b) {
        const u64 upper = edge[b >> Q], lower = edge[(b >> Q) + 1u];
        const u64 down = (u64)((b & ((1u << Q) - 1u)) + 1u) << shift(upper, lower);
        return upper - lower > down ? upper - down : lower;
    }
};
// Edges from N - 1 entries, one per thread from thread 1 on (in any order), and the two ends.  Contains three barriers; edge may be
// written and read again after it.
template <int B>
__device__ __forceinline__ void make_edges(u64* edge, u64 mine, u64 best, u64 worst) {
    constexpr u32 N = SplitBins<B>::N;
    const u32 tid = threadIdx.x;
    if (tid >= 1u && tid < N) edge[tid] = mine;
    __syncthreads();
    u32 r = 1;
    if (tid >= 1u && tid < N) {
#pragma unroll 8
        for (u32 i = 1; i < N; ++i) r += (edge[i] > mine || (edge[i] == mine && i < tid)) ? 1u : 0u;
    }
    __syncthreads();
    if (tid >= 1u && tid < N) edge[r] = mine;
    if (tid == 0) {
        edge[0] = best + 1u;
        edge[N] = worst;
    }
    __syncthreads();
}

template <int B>
__device__ __forceinline__ void order_range(u64& mn, u64& mx, OrderShared<B>& sm) {
    const u32 lane = lane_id(), wave = threadIdx.x >> 6;
    mn = wave_reduce64(mn, MinOf());
    mx = wave_reduce64(mx, MaxOf());
    if (lane == 63u) { sm.red[2 * wave] = mn; sm.red[2 * wave + 1] = mx; }
    __syncthreads();
    if constexpr (B > 512) {  // (see sum_of_waves; eight waves' are read as quickly one by one)
        const u32 w = lane % (u32)(B / 64);
        mn = last_lane64(wave_reduce64(sm.red[2 * w], MinOf()));
        mx = last_lane64(wave_reduce64(sm.red[2 * w + 1], MaxOf()));
    } else {
        mn = sm.red[0];
        mx = sm.red[1];
#pragma unroll
        for (int w = 1; w < B / 64; ++w) {
            mn = mn < sm.red[2 * w] ? mn : sm.red[2 * w];
            mx = mx > sm.red[2 * w + 1] ? mx : sm.red[2 * w + 1];
        }
    }
}
template <int B>
__device__ __forceinline__ u32 order_shift(u64 range) {
    constexpr u32 kBits = 31u - (u32)__builtin_clz(4 * B);
    const u32 width = range ? 64u - (u32)__builtin_clzll(range) : 0u;
    return width > kBits ? width - kBits : 0u;
}
// h[0 .. 4 B): counts -> exclusive prefix sums; into sm.sp the bin that holds rank want - 1; into sm.flag a 1 if a bin whose
// order matters (`sorted`: any up to that one; else that one alone) has more than `crowd`.  Two barriers.
template <int B>
__device__ __forceinline__ void order_scan(u32* h, u32 want, u32 crowd, bool sorted, OrderShared<B>& sm) {
    const u32 tid = threadIdx.x;
    u32 c[4], s = 0;
    bool most = false;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        c[i] = h[4 * tid + i];
        s += c[i];
    }
    const u32 incl = block_scan<B>(s, sm.wsum);
    u32 r = incl - s;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        h[4 * tid + i] = r;
        const bool last = r < want && r + c[i] >= want;
        if (last) sm.sp = 4 * tid + i;
        most = most || (c[i] > crowd && (last || (sorted && r < want)));
        r += c[i];
    }
    if (most) sm.flag = 1u;
    __syncthreads();
}

// One more in hist[bin]; lanes whose bin is the first lane's add together where they are many.  (Most of a crowd falls into one bin, and a wave's adds to one word are made one after the
// other: keep_best of 10308 entries, a ramp with infinities, 20.6 us, so 13.9.)
__device__ __forceinline__ void count_alike(u32* hist, u32 bin) {
    const u32 first = __builtin_amdgcn_readfirstlane(bin);
    const u64 alike = ballot64(bin == first);
    const u32 n = (u32)__popcll(alike);
    if (n >= 12u && bin == first) {
        if (mbcnt64(alike) == 0u) atomicAdd(&hist[bin], n);
    } else {
        atomicAdd(&hist[bin], 1u);
    }
}

// buf[0 .. want) to the row's output, from rank0 on.
template <int DT, int B>
__device__ __forceinline__ void order_output(const Params& P, int row, const RowShape& rs, const OrderShared<B>& sm, u32 want, u32 rank0,
                                             const ListEntry& ent) {
    char* out_v = (char*)P.out_values + (size_t)row * (size_t)P.k * KeyOf<DT>::kBytes;
    long long* out_i = P.out_indices + (size_t)row * (size_t)P.k;
    for (u32 i = threadIdx.x; i < want; i += B) {
        const u64 v = sm.buf[i];
        const u32 idx = ent.idx(v);
        out_i[rank0 + i] = (long long)idx;
        store_value<DT>(out_v, rank0 + i, raw_of_key<DT>(ent.key(v), idx, rs, P.dirmask));
    }
}

// C entries, load(0) .. load(C - 1) (1 <= C <= 8 B), which are the row's ranks rank0 .. rank0 + C - 1: write those below
// row_k to the output, in order if the call asked for that.  load() may read sm.buf.
// CUT: if a bin is crowded and the bins up to the one that rank k lies in have half the entries at most, those are put in order by themselves: their bins, divided
// again, are even as a rule (16-bit keys that rise along the row: some hundred neighbours to a value).  For k_list_finish, one row of 2^21 fp16 keys, a ramp, 4438 entries:
// k = 16, between splitters 52.2 us, so 42.5; k = 1, 48.0 / 38.9.
// PART: where no more than half of the entries lie in the bins that matter, those are spread over the threads anew once they are in place, one or two to a thread instead of a few in each of
// up to eight rounds that most waves have to go through; and who is alone in its bin has nothing to read.  One row of 2^24 fp32 keys, 6500 entries, k = 256, 32.0 us, so 30.3; of 2^20,
// k = 3000, 24.0 / 21.5.  171 rows of 223482 fp16 keys, k = 512, 37.8 / 35.8.  Where few waves order short lists it adds 0.1 us (300 rows of
// 30011 fp16 keys, k = 100, 15.25 / 15.4), and to 1024 rows of 2^17 bf16 keys, k = 1024, of which nearly all is wanted, 0.3.
template <int DT, int B, bool CUT = false, bool PART = CUT || B >= 512, class Load>
__device__ __forceinline__ void order_in_lds(const Params& P, int row, const RowShape& rs, OrderShared<B>& sm, u32 C, u32 rank0,
                                             Load&& load) {
    u32 tid = threadIdx.x;
    asm volatile("" : "+v"(tid));  // (what follows from it is worked out here and not kept for the whole kernel: k_list_row by 256 threads 95 registers, 102 without, four waves to a SIMD and not five)
    const u32 want = rs.k - rank0 < C ? rs.k - rank0 : C;
    const bool sorted = (P.flags & RTOPK_FLAG_SORTED) != 0u;
    const ListEntry ent = list_entry<DT>(P);
    u64 e[8], mn = ~0ull, mx = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        e[j] = 0;
        if ((u32)j * B < C) {  // (the same for the whole workgroup; lanes beyond the end read the last entry)
            const u32 i = tid + (u32)j * B;
            e[j] = load(i < C ? i : C - 1u);
        }
    }
    for (u32 j = tid; j <= 4u * B; j += B) sm.hist[j] = 0;
    if (tid == 0) sm.flag = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if ((u32)j * B < C) {
            mn = mn < e[j] ? mn : e[j];
            mx = mx > e[j] ? mx : e[j];
        }
    }
    order_range<B>(mn, mx, sm);
    const u32 sh = order_shift<B>(mx - mn);
#pragma unroll
    for (int j = 0; j < 8; ++j)
        if (tid + (u32)j * B < C) atomicAdd(&sm.hist[(u32)((mx - e[j]) >> sh) + 1u], 1u);  // (the bins' counts, one place up)
    __syncthreads();
    const u32 per = (C + (u32)B - 1u) / (u32)B;  // entries per thread
    order_scan<B>(sm.hist + 1, want, per < 4u ? kOrderCrowd / per : kOrderCrowd / 4u, sorted, sm);
    // entry j's rank, if it is wanted, among the entries of its bin, which are buf[from .. to); then every one to its place
    u32 left = C;  // (this many entries are spread over the threads)
    auto rank_and_place = [&](auto&& from, auto&& to) __attribute__((always_inline)) {
        u32 rank[4];  // two to a word
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            u32 r = 0xffffu;
            if ((u32)j * B < left && e[j] != ~0ull) {
                const u32 s0 = from(j), s1 = to(j);
                r = s0;
#pragma unroll 1
                for (u32 i = PART && s1 - s0 == 1u ? s1 : s0; i < s1; i += 4u) {  // (alone in its bin: nothing to read)
                    u64 b[4];
#pragma unroll
                    for (u32 x = 0; x < 4u; ++x) b[x] = sm.buf[i + x];
#pragma unroll
                    for (u32 x = 0; x < 4u; ++x) r += (b[x] > e[j] && i + x < s1) ? 1u : 0u;
                }
            }
            rank[j / 2] = (j & 1) ? rank[j / 2] | r << 16 : r;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const u32 r = (j & 1) ? rank[j / 2] >> 16 : rank[j / 2] & 0xffffu;
            if (r < want) sm.buf[r] = e[j];
        }
    };
    if (sm.flag == 0u) {
        // hist[b + 1]: where bin b begins, and once its entries are in place, where it ends; hist[b] is then where it begins
        const u32 last = sm.sp;  // (nothing beyond this bin is wanted)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const u32 bin = (u32)((mx - e[j]) >> sh);
            const bool is = tid + (u32)j * B < C && bin <= last;
            if (is) sm.buf[atomicAdd(&sm.hist[bin + 1u], 1u)] = e[j];
            if (!is || (!sorted && bin < last)) e[j] = ~0ull;  // (not an entry: those have at most 63 bits; nothing left to do with it)
        }
        __syncthreads();
        const u32 end = sm.hist[last + 1u];
        if (PART && per > 1u && end * 2u <= C) {
            const u32 first = sorted ? 0u : sm.hist[last];
            left = end;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                e[j] = ~0ull;
                if ((u32)j * B < end) {
                    const u32 i = tid + (u32)j * B;
                    if (i >= first && i < end) e[j] = sm.buf[i];
                }
            }
        }
        rank_and_place([&](int j) { return sm.hist[(u32)((mx - e[j]) >> sh)]; }, [&](int j) { return sm.hist[(u32)((mx - e[j]) >> sh) + 1u]; });
        __syncthreads();
        order_output<DT, B>(P, row, rs, sm, want, rank0, ent);
        return;
    }
    if constexpr (CUT) {
        const u32 last = sm.sp, end = last + 1u < 4u * B ? sm.hist[last + 2u] : C;
        __syncthreads();
        if (end * 2u <= C && end <= 8u * 256u) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const u32 bin = (u32)((mx - e[j]) >> sh);
                if (tid + (u32)j * B < C && bin <= last) sm.buf[atomicAdd(&sm.hist[bin + 1u], 1u)] = e[j];
            }
            __syncthreads();
            if (tid < 256u) order_in_lds<DT, 256>(P, row, rs, *(OrderShared<256>*)&sm, end, rank0, [&](u32 i) __attribute__((always_inline)) { return sm.buf[i]; });
            return;
        }
    }
    // crowded: bins between splitters, which are taken from the entries at equal distances (8 us; two entries per thread are through
    // the network in less)
    typedef SplitBins<B> Split;
    __syncthreads();  // (everybody has seen the flag)
    u32 at[8];  // bin, and which of its entries this one is
    if (per > 2u) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (tid + (u32)j * B < C) sm.buf[tid + (u32)j * B] = e[j];
        for (u32 j = tid; j < 4u * B + 2u; j += B) sm.hist[j] = 0;
        if (tid == 0) sm.flag = 0;
        __syncthreads();
        const u64 mine = tid < (u32)Split::N ? sm.buf[(u32)((u64)tid * C / (u32)Split::N)] : 0ull;
        __syncthreads();
        make_edges<B>(sm.buf, mine, mx, mn);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            at[j] = 0;
            if (tid + (u32)j * B < C) {
                const u32 bin = Split::bin(sm.buf, e[j]);
                at[j] = bin << 16 | atomicAdd(&sm.hist[bin], 1u);
            }
        }
        __syncthreads();
        order_scan<B>(sm.hist, want, kSplitCrowd, sorted, sm);
    }
    if (sm.flag == 0u) {
        const u32 last = sm.sp;
        if (tid == 0) sm.hist[4 * B] = C;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const u32 bin = at[j] >> 16;
            const bool is = tid + (u32)j * B < C && bin <= last;
            if (is) sm.buf[sm.hist[bin] + (at[j] & 0xffffu)] = e[j];
            if (!is || (!sorted && bin < last)) e[j] = ~0ull;
        }
        __syncthreads();
        rank_and_place([&](int j) { return sm.hist[at[j] >> 16]; }, [&](int j) { return sm.hist[(at[j] >> 16) + 1u]; });
    } else {
        u32 m = 64;
        while (m < C) m <<= 1;
        // (the network sorts upwards: complements; padding sorts last)
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (tid + (u32)j * B < C) sm.buf[tid + (u32)j * B] = ~e[j];
        for (u32 i = C + tid; i < m; i += B) sm.buf[i] = ~0ull;
        bitonic_sort<B>(sm.buf, m, tid);
        __syncthreads();
        for (u32 i = tid; i < want; i += B) sm.buf[i] = ~sm.buf[i];
    }
    __syncthreads();
    order_output<DT, B>(P, row, rs, sm, want, rank0, ent);
}

// The same for `count` entries at positions rank0 .. of list array `which`, however many: what LDS does not hold is
// first spread over bins in the other array (same positions; the bins divide the range evenly, so this ends after a
// few levels at most), and runs of bins of about 4 B entries are then taken one after the other.  `stack`: room for
// count / B + 16 records of this workgroup's own.
struct OrderRange { u32 at, count, which, pad; };
template <int DT, int B>
__device__ __forceinline__ void order_entries(const Params& P, int row, const RowShape& rs, OrderShared<B>& sm, u32 rank0, u32 count, u32 which,
                              OrderRange* stack) {
    constexpr u32 kCap = 8 * B;
    const u32 tid = threadIdx.x;
    u32 sp = 0;  // records on the stack (uniform)
    OrderRange cur{rank0, count, which, 0u};
    for (;;) {
        const u64* src = list_array(P, cur.which, row) + cur.at;
        __syncthreads();
        if (cur.count == 0) {  // (an empty bin and a large one that begin at the same rank)
        } else if (cur.count <= kCap) {
            order_in_lds<DT, B>(P, row, rs, sm, cur.count, cur.at, [&](u32 i) __attribute__((always_inline)) { return src[i]; });
        } else {
            u64* dst = list_array(P, 1u - cur.which, row) + cur.at;
            for (u32 j = tid; j < 4u * B; j += B) sm.hist[j] = 0;
            u64 mn = ~0ull, mx = 0;
#pragma unroll 1
            for (u32 i = tid; i < cur.count; i += B) {
                const u64 e = src[i];
                mn = mn < e ? mn : e;
                mx = mx > e ? mx : e;
            }
            order_range<B>(mn, mx, sm);  // (its barrier also covers the clearing)
            const u32 sh = order_shift<B>(mx - mn);
#pragma unroll 1
            for (u32 i = tid; i < cur.count; i += B) atomicAdd(&sm.hist[(u32)((mx - src[i]) >> sh)], 1u);
            __syncthreads();
            const u32 want = rs.k - cur.at < cur.count ? rs.k - cur.at : cur.count;
            order_scan<B>(sm.hist, want, ~0u, false, sm);
            const u32 end = (sm.sp + 1u < 4u * B) ? sm.hist[sm.sp + 1u] : cur.count;  // what begins below `want` ends here
            // runs of bins: a run begins at the first bin that starts beyond the next multiple of run_len, and at a bin
            // that alone holds more than run_len (so a run is one bin, whose range is a small part of this one, or
            // has at most 2 run_len entries: every round is strictly smaller than the one before)
            u32 run_len = kCap / 2u;
            while ((u64)run_len * (kCap / 2u) < (u64)cur.count) run_len *= 2u;  // (the list of beginnings fits sm.buf)
            u32 begins = 0, mask = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const u32 b = 4 * tid + i, s = sm.hist[b];
                const u32 n1 = b + 1u < 4u * B ? sm.hist[b + 1u] : cur.count;
                const bool first = s < want && (b == 0 || s / run_len > sm.hist[b - 1] / run_len || n1 - s > run_len);
                mask |= (first ? 1u : 0u) << i;
                begins += first ? 1u : 0u;
            }
            u32 slot = block_scan<B>(begins, sm.wsum) - begins;  // (and everybody has read sm.sp)
            u32* beg = (u32*)sm.buf;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if ((mask >> i) & 1u) beg[slot++] = sm.hist[4 * tid + i];
            if (tid == B - 1) sm.sp = slot;
            __syncthreads();
            const u32 nrun = sm.sp;
            for (u32 i = tid; i < nrun; i += B) {
                const u32 b = beg[i], n1 = i + 1 < nrun ? beg[i + 1] : end;
                stack[sp + i] = OrderRange{cur.at + b, n1 - b, 1u - cur.which, 0u};
            }
            __syncthreads();
#pragma unroll 1
            for (u32 i = tid; i < cur.count; i += B) {
                const u64 e = src[i];
                dst[atomicAdd(&sm.hist[(u32)((mx - e) >> sh)], 1u)] = e;
            }
            sp += nrun;
        }
        __syncthreads();
        if (sp == 0) return;
        cur = stack[--sp];
    }
}

// sm.buf[0 .. total), at most 8 B entries, into the output, by as few waves as hold them (barriers).  Begins with a barrier.
template <int DT, int B>
__device__ __forceinline__ void order_list(const Params& P, int row, const RowShape& rs, OrderShared<B>& sm, u32 total) {
    __syncthreads();
    auto listed = [&](u32 i) __attribute__((always_inline)) { return sm.buf[i]; };
    if (B > 256 && total <= 8u * 256u) {
        if (threadIdx.x >= 256u) return;
        order_in_lds<DT, 256, true>(P, row, rs, *(OrderShared<256>*)&sm, total, 0u, listed);
    } else if (B > 512 && total <= 8u * 512u) {
        if (threadIdx.x >= 512u) return;
        order_in_lds<DT, 512, true>(P, row, rs, *(OrderShared<512>*)&sm, total, 0u, listed);
    } else {
        order_in_lds<DT, B, true>(P, row, rs, sm, total, 0u, listed);
    }
}

// Where a list's entries are: one by one, a wave's at a time, and all of them -- f(entry, of(entry)) by the B threads, AHEAD loads in flight per thread (and as many chains of what `of` looks
// up in LDS).
struct EntriesAt {  // all together
    const u64* p;
    __device__ __forceinline__ u64 operator()(u32 i) const { return p[i]; }
    template <int B, u32 AHEAD, class Of, class F>
    __device__ __forceinline__ void each(u32 count, Of&& of, F&& f) const {
#pragma unroll 1
        for (u32 i = threadIdx.x; i < count; i += AHEAD * B) {  // (beyond the end: the last entry, which is not looked at)
            u64 e[AHEAD];
#pragma unroll
            for (u32 j = 0; j < AHEAD; ++j) e[j] = p[i + j * B < count ? i + j * B : count - 1u];
            u32 x[AHEAD];
#pragma unroll
            for (u32 j = 0; j < AHEAD; ++j) x[j] = of(e[j]);
#pragma unroll
            for (u32 j = 0; j < AHEAD; ++j)
                if (i + j * B < count) f(e[j], x[j]);
        }
    }
    template <u32 N>
    __device__ __forceinline__ void fetch(const u32 (&i)[N], u32, u32, u64 (&e)[N]) const {
#pragma unroll
        for (u32 j = 0; j < N; ++j) e[j] = p[i[j]];
    }
};
// In segments, of which begin[a] (in LDS, of at most MOST; ~0 or the list's length behind them) is the first entry's number: the first `slots` of a segment's entries at `front`, all of
// them in their places from `list` on, place[a] being how far those are from their numbers.  piece[a]: how many pieces of kPiece entries the segments before it have; piece[G]: all.
template <u32 MOST>
struct EntriesInSegments {
    static constexpr u32 kPiece = 256;
    const u64 *front, *list;
    const u32 *begin, *place, *piece;
    u32 slots, G;
    __device__ __forceinline__ u64 at(u32 a, u32 i) const {
        const u32 l = i - begin[a];
        return *(l < slots ? front + (a * slots + l) : list + (place[a] + i));
    }
    // (No branches: eight entries' searches and loads are under way together.  With loops that end when they have found it, and segments' places worked out for every entry,
    // one row of 2^20 fp32 keys, a ramp, k = 3000, took 81.7 us, so 71.2; 16 of 2^24, k = 512, of which nothing is too long, 38.6 / 38.0.)
    __device__ __forceinline__ u64 operator()(u32 i) const {
        u32 a = 0;  // the segment that holds entry i: the last one that begins at or before it
#pragma unroll
        for (u32 step = MOST / 2u; step > 0; step /= 2u) a += begin[a + step] <= i ? step : 0u;
        return at(a, i);
    }
    // A wave's entries i[.], all of them in [i0, i1].  Lists that are far too long lie in few long segments: those of the ends are counted by all lanes together, and what is left
    // to be searched between them is a step or two, as a rule none.
    template <u32 N>
    __device__ __forceinline__ void fetch(const u32 (&i)[N], u32 i0, u32 i1, u64 (&e)[N]) const {
        u32 a0 = 0, a1 = 0;
#pragma unroll
        for (u32 j = 0; j < MOST / 64u; ++j) {
            const u32 b = begin[j * 64u + lane_id()];
            a0 += (u32)__popcll(ballot64(b <= i0));
            a1 += (u32)__popcll(ballot64(b <= i1));
        }
        --a0;  // (begin[0] is 0)
        --a1;
        u32 a[N];
#pragma unroll
        for (u32 j = 0; j < N; ++j) a[j] = a0;
#pragma unroll 1
        for (u32 step = a1 > a0 ? 1u << (31u - (u32)__builtin_clz(a1 - a0)) : 0u; step > 0; step /= 2u) {
#pragma unroll
            for (u32 j = 0; j < N; ++j) {
                const u32 m = a[j] + step;
                a[j] = m <= a1 && begin[m < a1 ? m : a1] <= i[j] ? m : a[j];
            }
        }
#pragma unroll
        for (u32 j = 0; j < N; ++j) e[j] = at(a[j], i[j]);
    }
    // A wave takes every B / 64-th piece, the next one's loads under way: the segment of a piece is the same for all lanes, and 64 pieces' segments are searched for at once.  (An entry's
    // segment searched for by its lane, 50 instructions: 53440 entries in 18.5 us.)
    template <int B, u32 AHEAD, class Of, class F>
    __device__ __forceinline__ void each(u32, Of&& of, F&& f) const {
        static_assert(kPiece == 64u * AHEAD, "a piece is what a wave has in flight");
        constexpr u32 W = (u32)B / 64u;
        const u32 lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), pieces = __builtin_amdgcn_readfirstlane(piece[G]);
#pragma unroll 1
        for (u32 q0 = wave; q0 < pieces; q0 += 64u * W) {
            const u32 left = (pieces - q0 + W - 1u) / W, n = left < 64u ? left : 64u;
            const u32 q = q0 + W * (lane < n ? lane : n - 1u);
            u32 mine = 0;
#pragma unroll
            for (u32 step = MOST / 2u; step > 0; step /= 2u) mine += piece[mine + step] <= q ? step : 0u;
            const u32 l0 = (q - piece[mine]) * kPiece, rest = begin[mine + 1u] - begin[mine] - l0, there = place[mine] + begin[mine];
            auto load = [&](u32 t, u64 (&e)[AHEAD]) __attribute__((always_inline)) {
                const u32 a = (u32)__builtin_amdgcn_readlane((int)mine, (int)t), l = (u32)__builtin_amdgcn_readlane((int)l0, (int)t);
                const u32 c = (u32)__builtin_amdgcn_readlane((int)rest, (int)t);
                const u64 *head = front + a * slots, *tail = list + (u32)__builtin_amdgcn_readlane((int)there, (int)t);
#pragma unroll
                for (u32 j = 0; j < AHEAD; ++j) {
                    if (j * 64u >= c) break;
                    const u32 i = l + (j * 64u + lane < c ? j * 64u + lane : c - 1u);
                    e[j] = *((i < slots ? head : tail) + i);
                }
            };
            auto use = [&](u32 t, const u64 (&e)[AHEAD]) __attribute__((always_inline)) {
                const u32 c = (u32)__builtin_amdgcn_readlane((int)rest, (int)t);
                u32 x[AHEAD];
#pragma unroll
                for (u32 j = 0; j < AHEAD; ++j) x[j] = of(e[j]);
#pragma unroll
                for (u32 j = 0; j < AHEAD; ++j)
                    if (j * 64u + lane < c) f(e[j], x[j]);
            };
            u64 e[2][AHEAD] = {};
            load(0, e[0]);
#pragma unroll 1
            for (u32 t = 0; t < n; t += 2u) {
                if (t + 1u < n) load(t + 1u, e[1]);
                use(t, e[0]);
                if (t + 2u < n) load(t + 2u, e[0]);
                if (t + 1u < n) use(t + 1u, e[1]);
            }
        }
    }
};

// Those of src's `count` entries that lie in [lo, hi) to buf; returns how many there are (up to 8 B are kept).  Begins and ends with a barrier.
template <int B, u32 kAhead, class Src>
__device__ __forceinline__ u32 order_gather(const Src& src, u32 count, u64 lo, u64 hi, OrderShared<B>& sm, u32* run) {
    const u32 tid = threadIdx.x;
    __syncthreads();
    if (tid == 0) *run = 0;
    __syncthreads();
    src.template each<B, kAhead>(count, [](u64) { return 0u; }, [&](u64 e, u32) __attribute__((always_inline)) {
        if (e >= lo && e < hi) {
            const u32 at = atomicAdd(run, 1u);
            if (at < 8u * B) sm.buf[at] = e;
        }
    });
    __syncthreads();
    return *run;
}

// The entries of src in [lo, hi), which are the row's ranks from rank0 on, a chunk that LDS holds after the other; where the
// chunk ends is found by dividing the range evenly, as often as it takes (entries are distinct).
template <int DT, int B, u32 kAhead, class Src>
__device__ __forceinline__ void order_in_chunks(const Params& P, int row, const RowShape& rs, OrderShared<B>& sm, const Src& src, u32 count,
                                                u32 rank0, u64 lo, u64 hi, u32* run) {
    const u32 tid = threadIdx.x;
    while (hi > lo && rank0 < rs.k) {
        u64 a = lo, cut;
        for (;;) {
            const u32 sh = order_shift<B>(hi - a - 1u);
            __syncthreads();
            for (u32 j = tid; j < 4u * B; j += B) sm.hist[j] = 0;
            if (tid == 0) sm.sp = 4u * B;
            __syncthreads();
            src.template each<B, kAhead>(count, [](u64) { return 0u; }, [&](u64 e, u32) __attribute__((always_inline)) {
                if (e >= a && e < hi) atomicAdd(&sm.hist[(u32)((hi - 1u - e) >> sh)], 1u);
            });
            __syncthreads();
            order_scan<B>(sm.hist, 8u * B + 1u, ~0u, false, sm);  // sp: the first bin whose end lies beyond 8 B entries
            const u32 bins = sm.sp;
            const u64 down = (u64)bins << sh;
            cut = bins < 4u * B && hi - a > down ? hi - down : a;
            if (bins != 0u) break;
            if (hi - a > (1ull << sh)) a = hi - (1ull << sh);
        }
        const u32 n = order_gather<B, kAhead>(src, count, cut, hi, sm, run);
        if (n != 0u) order_in_lds<DT, B>(P, row, rs, sm, n, rank0, [&](u32 i) __attribute__((always_inline)) { return sm.buf[i]; });
        rank0 += n;
        hi = cut;
    }
}

// One of `parts` workgroups that put src's `count` entries in order, the row's ranks from rank0 on.  Each reads all of it once and counts
// it into bins between splitters, which are entries at equal distances, so that all of them see the same bins; runs of bins that LDS
// holds are dealt to them, and each reads all of it again for every run of its own.  Nobody waits for anybody and
// nothing is moved in memory.  One workgroup reads about 0.1 TB/s, so 2^20 entries take 256 of them about 0.2 ms.
constexpr u32 kOrderRuns = 128;  // runs that a workgroup notes at a time
template <int B>
struct OrderParts {
    u64 edge[SplitBins<B>::N + 1];
    u64 lo[kOrderRuns], hi[kOrderRuns];
    u32 start[kOrderRuns], size[kOrderRuns];
    u32 nrun, run;
};
template <int DT, int B, class Src>
__device__ __forceinline__ void order_shared(const Params& P, int row, const RowShape& rs, OrderShared<B>& sm, OrderParts<B>& sp, const Src& src,
                                             u32 count, u32 rank0, u32 part, u32 parts) {
    typedef SplitBins<B> Split;
    constexpr u32 kCap = 8 * B, kRun = kCap * 3 / 4, kBig = kCap / 4, kAhead = 4;  // (registers)
    const u32 tid = threadIdx.x, want = rs.k - rank0 < count ? rs.k - rank0 : count;
    __syncthreads();
    // Little is wanted of much: a bound from 8 B entries at equal distances, and one pass that gathers what is not below it.
    {
        const float ks = (float)want * ((float)kCap / (float)count);
        const u32 rank = (u32)(ks + 5.0f * __builtin_sqrtf(ks) + 5.0f);
        if (count > kCap && (u64)rank * count < (u64)kCap * (kCap / 8u * 7u)) {
            if (part != 0u) return;
            u64 e[8], lo = ~0ull, hi = 0;
            {
                const u32 first = __builtin_amdgcn_readfirstlane(tid >> 6) * 512u;
                u32 i[8];
#pragma unroll
                for (u32 j = 0; j < 8; ++j) i[j] = (u32)((u64)(first + j * 64u + lane_id()) * count / kCap);
                src.template fetch<8>(i, (u32)((u64)first * count / kCap), (u32)((u64)(first + 511u) * count / kCap), e);
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                lo = lo < e[j] ? lo : e[j];
                hi = hi > e[j] ? hi : e[j];
            }
            order_range<B>(lo, hi, sm);
            u32 left = rank;
            for (;;) {  // [lo, hi] holds the entry in question
                const u32 sh = order_shift<B>(hi - lo);
                __syncthreads();
                for (u32 j = tid; j < 4u * B; j += B) sm.hist[j] = 0;
                __syncthreads();
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (e[j] >= lo && e[j] <= hi) count_alike(sm.hist, (u32)((hi - e[j]) >> sh));
                __syncthreads();
                order_scan<B>(sm.hist, left, ~0u, false, sm);
                const u32 b = sm.sp, s0 = sm.hist[b], inside = b + 1u < 4u * B ? sm.hist[b + 1u] - s0 : 0u;
                left -= s0;
                hi -= (u64)b << sh;
                lo = hi - lo > (1ull << sh) - 1u ? hi - ((1ull << sh) - 1u) : lo;
                if (sh == 0u || (b + 1u < 4u * B && inside <= 4u + rank / 8u)) break;
            }
            const u32 n = order_gather<B, kAhead>(src, count, lo, ~0ull, sm, &sp.run);
            if (n >= want && n <= kCap) {
                order_in_lds<DT, B>(P, row, rs, sm, n, rank0, [&](u32 i) __attribute__((always_inline)) { return sm.buf[i]; });
                return;
            }
            __syncthreads();
            parts = 1;  // (an unlucky draw: everything, alone)
        }
    }
    if (count <= kCap) {
        if (part == 0u) order_in_lds<DT, B>(P, row, rs, sm, count, rank0, [&](u32 i) __attribute__((always_inline)) { return src(i); });
        return;
    }
    // (the ends: nothing is known of the best and the worst entry but that they are entries)
    const u64 end = list_entry<DT>(P).end();
    make_edges<B>(sp.edge, tid < (u32)Split::N ? src((u32)((u64)tid * count / (u32)Split::N)) : 0ull, end - 1u, 0ull);
    for (u32 done = 0;;) {
        for (u32 j = tid; j < 4u * B + 2u; j += B) sm.hist[j] = 0;
        __syncthreads();
        src.template each<B, kAhead>(count, [&](u64 e) __attribute__((always_inline)) { return Split::bin(sp.edge, e); },
                      [&](u64, u32 bin) __attribute__((always_inline)) { atomicAdd(&sm.hist[bin], 1u); });
        __syncthreads();
        order_scan<B>(sm.hist, want, ~0u, false, sm);
        if (tid == 0) sm.hist[4 * B] = count;
        __syncthreads();
        // A run begins at the first bin beyond a multiple of kRun, and at and after a bin of more than kBig: so it is such a bin
        // or has at most kRun + kBig entries.
        u32 begins = 0, mask = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const u32 b = 4 * tid + i, s = sm.hist[b], before = b == 0u ? 0u : sm.hist[b - 1];
            const bool first = s < want && (b == 0u || s / kRun != before / kRun || sm.hist[b + 1] - s > kBig || s - before > kBig);
            mask |= (first ? 1u : 0u) << i;
            begins += first ? 1u : 0u;
        }
        u32 slot = block_scan<B>(begins, sm.wsum) - begins;
        const u32 last = sm.sp;
        u32* first_bin = (u32*)sm.buf;  // of every run (nothing else is there yet)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if ((mask >> i) & 1u) first_bin[slot++] = 4 * tid + i;
        if (tid == B - 1) sp.nrun = slot;
        __syncthreads();
        const u32 nrun = sp.nrun;
        // this workgroup's next runs: part, part + parts, ...
        for (u32 i = tid; i < kOrderRuns; i += B) {
            const u64 r64 = (u64)part + (u64)(done + i) * parts;
            if (r64 < nrun) {
                const u32 r = (u32)r64, b0 = first_bin[r], b1 = r + 1u < nrun ? first_bin[r + 1u] - 1u : last;
                sp.hi[i] = b0 == 0u ? end : Split::floor_of(sp.edge, b0 - 1u);
                sp.lo[i] = Split::floor_of(sp.edge, b1);
                sp.start[i] = sm.hist[b0];
                sp.size[i] = sm.hist[b1 + 1u] - sm.hist[b0];
            }
        }
        __syncthreads();
        for (u32 i = 0; i < kOrderRuns; ++i) {
            if ((u64)part + (u64)(done + i) * parts >= nrun) return;
            const u32 n = sp.size[i], r0 = rank0 + sp.start[i];
            if (n > kCap) {
                order_in_chunks<DT, B, kAhead>(P, row, rs, sm, src, count, r0, sp.lo[i], sp.hi[i], &sp.run);
            } else if (n != 0u) {
                order_gather<B, kAhead>(src, count, sp.lo[i], sp.hi[i], sm, &sp.run);
                order_in_lds<DT, B>(P, row, rs, sm, n, r0, [&](u32 i) __attribute__((always_inline)) { return sm.buf[i]; });
            }
        }
        done += kOrderRuns;
        __syncthreads();
    }
}

// ------------------------------------------------------------------------------------------------
// short lists
// ------------------------------------------------------------------------------------------------

// One row's record: how many were listed, all ranked directly.
__device__ __forceinline__ void list_record(rtopk_row_trace* st, const RowShape& rs, u32 listed, u32 where) {
    st->pass_rec[0].bin = 0;
    st->pass_rec[0].k_after = 0;
    st->pass_rec[0].cand_after = 0;
    st->pass_rec[0].winners = rs.k;
    st->pass_rec[0].out_before = 0;
    st->pass_rec[0].cand_before = listed;
    st->pass_rec[0].window = SRC_RANK;
    st->pass_rec[0].where = where;
    st->pre_kept = listed;
}

template <int DT>
__device__ __forceinline__ u64 src_vectors(const RowShape& rs) {
    KeySource<DT, 64, 4, false> src;
    src.init(rs);
    return src.nvec;
}
// Elements that equal T, by tile.  (Counted by atomics: read past the vector cache, which does not see those.)
struct TileCounts {
    const u32* te;
    __device__ __forceinline__ u32 operator()(u32 i) const { return __hip_atomic_load(&te[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
};
// Elements equal to T, lowest positions first, to the output behind the `listed` better ones.  Workgroup w of nw takes the
// tiles w, w + nw, ... as far as they are needed.  te(i): how many tile i has.  Returns false if the row has too few of them.
template <int DT, int B, class Source, class Counts>
__device__ __forceinline__ bool ties_of_row(const Params& P, Counts&& te, int row, const RowShape& rs, u32 listed, u32 T, u32 w, u32 nw,
                            u32* before, u32* wsum) {
    constexpr u32 E = Source::E, kStep = 2;
    static_assert(Source::kTileVecs % (kStep * B) == 0, "whole steps");
    Source src;
    src.init(rs);
    const u32 ntiles = src.ntiles(), tid = threadIdx.x, want = rs.k - listed;
    char* out_v = (char*)P.out_values + (size_t)row * (size_t)P.k * KeyOf<DT>::kBytes;
    long long* out_i = P.out_indices + (size_t)row * (size_t)P.k;
    u32 base = 0;  // equal elements in the tiles before this block of B tiles
    for (u32 t0 = 0; t0 < ntiles; t0 += B) {
        const u32 c = t0 + tid < ntiles ? te(t0 + tid) : 0u;
        __syncthreads();
        const u32 incl = block_scan<B>(c, wsum);
        before[tid] = base + incl - c;
        if (tid == B - 1) before[B] = base + incl;
        __syncthreads();
        const u32 next = before[B];
        for (u32 k = (w + nw - t0 % nw) % nw; k < (u32)B && t0 + k < ntiles; k += nw) {
            const u32 at = before[k];
            if (at >= want) break;
            if (before[k + 1] == at) continue;
            // this tile, in steps of kStep neighbouring vectors per thread, so that thread order is index order
            u32 begin = at;
            for (u32 v0 = 0; v0 < (u32)Source::kTileVecs; v0 += kStep * (u32)B) {
                const u64 v = (u64)(t0 + k) * Source::kTileVecs + v0 + (u64)tid * kStep;
                u32 hit = 0;
#pragma unroll
                for (u32 u = 0; u < kStep; ++u) {
                    uint4 q = v + u < src.nvec ? load16<false>(src.abase + (v + u)) : make_uint4(0, 0, 0, 0);
                    keys_of_vector<DT>(q, P.dirmask);
#pragma unroll
                    for (u32 j = 0; j < E; ++j) {
                        const bool is = (u32)(v + u) * E + j - src.lead < rs.n && key_in_vector<DT>(q, (int)j) == T;
                        hit |= (is ? 1u : 0u) << (u * E + j);
                    }
                }
                const u32 n = (u32)__builtin_popcount(hit);
                __syncthreads();  // (wsum's last readers are done)
                const u32 incl = block_scan<B>(n, wsum);
                u32 pos = begin + incl - n;
#pragma unroll
                for (u32 w = 0; w < (u32)(B / 64); ++w) begin += wsum[w];  // (the scan leaves every wave's sum there)
                for (; hit != 0u && pos < want; hit &= hit - 1u, ++pos) {
                    const u32 idx = (u32)v * E + (u32)__builtin_ctz(hit) - src.lead;
                    out_i[listed + pos] = (long long)idx;
                    store_value<DT>(out_v, listed + pos, raw_of_key<DT>(T, idx, rs, P.dirmask));
                }
            }
        }
        base = next;
        if (base >= want) return true;
        __syncthreads();
    }
    return false;
}

// e[j], ~0 where there is none: those that may be among the best `want`, at most 8 B, go to sm.buf, in any order; returns how many that are.  *crowd: the bins that divide
// the entries' range evenly had to be laid again, inside the one that rank want - 1 lies in, because it held too many.  (Entries are distinct: at some point it does not.  A row of
// 2^20 fp32 keys, a ramp with infinities, k = 1000, 10308 entries, which order_shared put in order otherwise, 57.4 us, so 51.0.)  Ends with a barrier.
template <int B, u32 N>
__device__ __forceinline__ u32 keep_best(const u64 (&e)[N], u32 total, u32 want, OrderShared<B>& sm, bool* crowd) {
    const u32 tid = threadIdx.x;
    u64 mn = ~0ull, mx = 0;
#pragma unroll
    for (u32 j = 0; j < N; ++j) {
        if (e[j] == ~0ull) continue;
        mn = mn < e[j] ? mn : e[j];
        mx = mx > e[j] ? mx : e[j];
    }
    order_range<B>(mn, mx, sm);
    u32 left = want, above = 0, inside = total;  // entries above mx, and from there down to mn
    *crowd = false;
#pragma unroll 1
    for (;;) {
        const u32 sh = order_shift<B>(mx - mn);
        for (u32 j = tid; j < 4u * B; j += B) sm.hist[j] = 0;
        __syncthreads();
#pragma unroll
        for (u32 j = 0; j < N; ++j)
            if (e[j] >= mn && e[j] <= mx) count_alike(sm.hist, (u32)((mx - e[j]) >> sh));
        __syncthreads();
        order_scan<B>(sm.hist, left, ~0u, false, sm);
        const u32 last = sm.sp, before = sm.hist[last], upto = last + 1u < 4u * B ? sm.hist[last + 1u] : inside;
        if (tid == 0) sm.flag = 0;
        __syncthreads();
        const u64 floor = mx - mn > ((u64)(last + 1u) << sh) - 1u ? mx - (((u64)(last + 1u) << sh) - 1u) : mn;
        if (above + upto <= 8u * B && (above + upto <= 2048u || above + upto <= want + want / 4u)) {
            mn = floor;
            above += upto;
            break;
        }
        mx -= (u64)last << sh;
        mn = floor;
        above += before;
        left -= before;
        inside = upto - before;
        *crowd = true;
    }
    // (a lane's places by the wave, a wave's by the workgroup: bins would be places, too, but not those of what lies above them)
#pragma unroll
    for (u32 j = 0; j < N; ++j) {
        const bool is = e[j] >= mn && e[j] != ~0ull;
        const u64 have = ballot64(is);
        if (have == 0) continue;
        u32 at = 0;
        if (lane_id() == 0) at = atomicAdd(&sm.flag, (u32)__popcll(have));
        at = __builtin_amdgcn_readfirstlane(at) + mbcnt64(have);
        if (is) sm.buf[at] = e[j];
    }
    __syncthreads();
    return above;
}

// ------------------------------------------------------------------------------------------------
// rows whose list was no use
// ------------------------------------------------------------------------------------------------
// One workgroup selects the row's k-th key from all of X (three or four sweeps), lists what is better, counts what
// is equal, and goes on as usual.
template <int DT, int B>
__device__ __forceinline__ u32 list_anew(const Params& P, const ListPlan& L, int row, const RowShape& rs, rtopk_row_trace* st,
                                         RankShared& rank, u32* run, u32* hist, u32* wsum) {
    typedef ListSource<DT, false> Source;
    constexpr u32 E = Source::E;
    const u32 tid = threadIdx.x, lane = lane_id();
    Source src;
    src.init(rs);
    const u32 nvec = (u32)src.nvec;
    constexpr u32 kAhead = 4;  // vectors in flight per thread
    auto fetch = [&](u32 b, uint4 (&q)[kAhead]) __attribute__((always_inline)) {  // (beyond the end: the last one, which is not looked at)
#pragma unroll
        for (u32 c = 0; c < kAhead; ++c) q[c] = load16<false>(src.abase + (b + c * B + tid < nvec ? b + c * B + tid : nvec - 1u));
#pragma unroll
        for (u32 c = 0; c < kAhead; ++c) keys_of_vector<DT>(q[c], P.dirmask);
    };
    bool exact;
    const u32 T = sample_rank<B>([&](auto&& f) __attribute__((always_inline)) {
#pragma unroll 1
        for (u32 b = 0; b < nvec; b += kAhead * B) {
            uint4 q[kAhead];
            fetch(b, q);
#pragma unroll
            for (u32 c = 0; c < kAhead; ++c) {
                const u32 v = b + c * B + tid;
#pragma unroll
                for (u32 j = 0; j < E; ++j)
                    if (v < nvec && v * E + j - src.lead < rs.n) f(key_in_vector<DT>(q[c], (int)j));
            }
        }
    }, rs.k, 0u, 0xffffffffu, rank, &exact);
    u32* te = list_part<u32>(P, row, L.tile_off);
    const u32 nt = src.ntiles();
    for (u32 j = tid; j < nt; j += B) te[j] = 0;
    if (tid == 0) *run = 0;
    __syncthreads();
    const ListEntry ent = list_entry<DT>(P);
    u64* list = list_array(P, 1u, row);
    const u32 room = (u32)((P.n + 1) / 2);
#pragma unroll 1
    for (u32 b = 0; b < nvec; b += kAhead * B) {  // (whole waves: a wave's 64 vectors lie in one tile)
        uint4 q[kAhead];
        fetch(b, q);
#pragma unroll
        for (u32 c = 0; c < kAhead; ++c) {
            const u32 v = b + c * B + tid;
            u32 eq = 0;
#pragma unroll
            for (u32 j = 0; j < E; ++j) {
                const u32 key = key_in_vector<DT>(q[c], (int)j), idx = v * E + j - src.lead;
                const bool valid = v < nvec && idx < rs.n;
                eq += valid && key == T ? 1u : 0u;
                if (valid && key > T) {
                    const u32 at = atomicAdd(run, 1u);
                    if (at < room) list[at] = ent.of(key, idx);
                }
            }
            eq = wave_inclusive_scan(eq);
            if (lane == 63u && eq != 0u) atomicAdd(&te[(v - 63u) / (u32)Source::kTileVecs], eq);
        }
    }
    __syncthreads();
    const u32 listed = *run;
    if (listed > room) {
        if (tid == 0) st->error |= 4u;  // never expected: little more than k are better than T
        return 0;
    }
    if (tid == 0) list_record(st, rs, listed, 5u);
    if (listed < rs.k) {
        __syncthreads();
        ties_of_row<DT, B, Source>(P, TileCounts{te}, row, rs, listed, T, 0u, 1u, hist, wsum);
        __syncthreads();
    }
    return listed;
}
// All that is missing afterwards is the order of the returned number of entries, in list array 1: fewer than k, so that a short list's are in LDS here (ord.buf).  Ends with a barrier.
template <int DT, int B, bool LONG>
__device__ __forceinline__ u32 redo_row(const Params& P, const ListPlan& L, int row, const RowShape& rs, rtopk_row_trace* st, u32 why,
                                        OrderShared<B>& ord, RankShared& rank, u32* run) {
    if (threadIdx.x == 0) {
        st->redo_why = why;
        st->redo |= kRedoRow;
    }
    __syncthreads();
    u32 count = list_anew<DT, B>(P, L, row, rs, st, rank, run, ord.hist, ord.wsum);
    __syncthreads();
    if constexpr (!LONG) {
        if (count > 8u * B) {  // never expected: k is less
            if (threadIdx.x == 0) st->error |= 4u;
            count = 0;
        }
        const u64* list = list_array(P, 1u, row);
        for (u32 i = threadIdx.x; i < count; i += B) ord.buf[i] = list[i];
        __syncthreads();
    }
    return __builtin_amdgcn_readfirstlane(count);
}

// The list of one row into the output.  Blocks [0, batch): a row each.  Blocks beyond: L.ties per row, for rows whose
// equal elements were counted.  A list that LDS does not hold is the one workgroup's, too: little of it is wanted, by the plan's own limit on k, and that takes one bound and
// one gathering pass, which nobody can share.  (So much is wanted that others could help in 16-bit rows of 1.3 to 1.5 million keys alone, k of 4097 to 4150, of which nearly half is listed; the sample would
// have to miss that.)
// Lists that are far too long (trends, blocks of equal neighbours), us, put in order by a kernel of their own, which every call then waited for / by this one, looked through entry by entry / so:
// 2^24 fp32 keys, blocks, k = 300, 46528 entries, 57 / 83 / 63; four rows of 2^20 fp16 keys, a ramp with infinities, k = 300, 50 / 81 / 53, by 512 threads (256: 70); 33 rows of 400000 fp32 keys, k = 300,
// 192572 entries, 275 / 1986 / 132.
// Bound by latency.  The first entries of every segment lie together (L.slots of each) and are read before it is known how many there are: a search by
// every entry for the segment that holds it, and 1024 segments all over the list array, took 6.2 us for 3300 entries; this 3.3 for 5800.  (Ordered from
// the registers they are read to, 16 places per thread, they need not be put together first, but every phase takes longer: 12 / 15.5 us in all.)
// STREAM: k_list_stream's lists, in as many segments as there are compute units.  (Told apart while it runs, one row of 2^24 fp32 keys, k = 256, 12.0 us; compiled apart 11.7.)
template <int DT, int B, bool STREAM>
__global__ void __launch_bounds__(B) k_list_finish(Params P, ListPlan L) {
    constexpr u32 kMost = 16;  // places per thread
    constexpr u32 kMostSegments = B < 1024 ? 256 : 512;
    __shared__ union { OrderShared<B> ord; RankShared rank; } lds;
    __shared__ OrderParts<B> shared;
    __shared__ u32 segs[B + 1], place[B], piece[B + 1];
    OrderShared<B>& sm = lds.ord;
    const u32 tid = threadIdx.x, G = (u32)L.G, slots = L.slots, log = 31u - (u32)__builtin_clz(slots);
    const bool for_ties = blockIdx.x >= (u32)P.batch;
    const int row = __builtin_amdgcn_readfirstlane(for_ties ? (int)((blockIdx.x - (u32)P.batch) / (u32)L.ties) : (int)blockIdx.x);
    const u32 places = G * slots;  // (at most kMost * B)
    const u64* front = list_part<u64>(P, row, L.front_off);
    // (k_list_sweep's few long segments: entries look for theirs, where the list is short, or so long that all waves are needed to order it.  One
    // row of 1048869 fp16 keys, k = 3990, 34.7 us, put together first 37.0; 41 fp32 rows of 74007, k = 28, 20.7 / 21.5; but eleven of 135112, k = 615, 24.9 / 22.5.)
    constexpr bool few = !STREAM;
    // (the lengths and the decision before the entries: what counts of a row with ties does not wait for the places)
    const uint2 seg = tid < G ? list_part<uint2>(P, row, L.seg_off)[tid] : make_uint2(0u, 0u);  // (G is at most B)
    const u32 c = seg.x;
    const ListRow* lr = list_row(P, row);
    const u32 mode = lr->mode;
    __builtin_amdgcn_sched_barrier(0);
    u64 e[kMost] = {};
    if (!for_ties && !(few && B <= 512)) {
#pragma unroll
        for (u32 j = 0; j < kMost; ++j) {
            if (tid + j * (u32)B < places) e[j] = front[tid + j * (u32)B];
        }
    }
    if (mode == kListSkip) return;
    const RowShape rs = row_shape_scalar<DT>(P, row);
    rtopk_row_trace* st = row_state(P, row);
    const u32 incl = block_scan<B>(c, sm.wsum);
    if (tid != G) segs[tid] = tid < G ? incl - c : ~0u;
    if (tid == B - 1) segs[G] = incl;
    const u32 unit = few ? (u32)ListSource<DT, false>::kTileVecs : kWaveVecs;
    if (few && tid < G) place[tid] = list_segment<DT>(rs, tid, G, unit) - (incl - c);
    // (as scalars: branches on what the compiler takes to differ by lane are laid one behind the other, with the entries in registers through all of them)
    const bool over = __builtin_amdgcn_readfirstlane(__syncthreads_or(c > slots + (few ? 8u : 0u) ? 1 : 0)) != 0;  // (a segment has more than its places, or many more)
    const u32 total = __builtin_amdgcn_readfirstlane(segs[G]);
    u32 equal = 0;  // elements that equal T, where they were counted
    if (mode == kListTied) {
        (void)block_scan<B>(seg.y, sm.wsum);
        equal = sum_of_waves<B>(sm.wsum, 1);
        __syncthreads();
    }
    const bool few_in_all = (u64)total + equal < (u64)rs.k, useless = few_in_all || total > (u32)((P.n + 1) / 2);
    const u64* from = list_array(P, 1u, row);
    const EntriesInSegments<kMostSegments> entry{front, from, segs, place, piece, slots, G};
    auto find_places = [&]() __attribute__((always_inline)) {  // (k_list_stream's, which are rarely needed)
        if (few) return;
        if (tid < G) place[tid] = list_segment<DT>(rs, tid, G, unit) - (incl - c);
        __syncthreads();
    };
    if (for_ties) {
        if (useless || mode != kListTied || total >= rs.k) return;
        const u32 w = (blockIdx.x - (u32)P.batch) % (u32)L.ties;
        const TileCounts tiles{list_part<u32>(P, row, L.tile_off)};
        constexpr u32 kParts = (u32)ListSource<DT, false>::kTileVecs / kWaveVecs;
        const u32 parts = (u32)((src_vectors<DT>(rs) + kWaveVecs - 1u) / kWaveVecs);
        auto count = [&](u32 i) __attribute__((always_inline)) {  // (k_list_stream's tiles are smaller)
            if (few) return tiles(i);
            u32 n = 0;
#pragma unroll
            for (u32 c = 0; c < kParts; ++c) n += kParts * i + c < parts ? tiles(kParts * i + c) : 0u;
            return n;
        };
        if (!ties_of_row<DT, B, ListSource<DT, false>>(P, count, row, rs, total, lr->T, w, (u32)L.ties, sm.hist, sm.wsum) && w == 0 && tid == 0)
            st->error |= 4u;  // never expected: there are enough of them
        return;
    }
    u32 n = total;
    if (!useless && tid == 0) list_record(st, rs, total, 5u);
    if (total == 0 && !useless) return;
    // (A list that LDS does not hold, though not much longer than expected, is cut down first.  Not every one that is much longer than what is wanted of it: 5800 entries, k = 256, 12.0 / 15.8 us.)
    // (512 threads: what is longer than four per thread is not what the plan expects, and a crowd as a rule.  16 rows of 2^20 fp16 keys, a ramp, k = 40, 2936 entries: ordered whole 47.1, cut down first 35.8.)
    constexpr u32 kWhole = B <= 512 ? 4u * B : 8u * B;  // (L.room)
    if (few && !useless && (B <= 512 || total > 4096u) && total <= kWhole) {
        order_in_lds<DT, B, false, true>(P, row, rs, sm, total, 0u, entry);
        return;
    }
    // (What is rarely there to be done lies in one place: among the usual steps it costs them 0.3 to 1 us of fetching instructions.)
    if (__builtin_expect(useless || total > kWhole, 0)) {
        if (useless) {
            n = redo_row<DT, B, false>(P, L, row, rs, st, few_in_all ? 8u : 5u, sm, lds.rank, &shared.run);
            if (n == 0u) return;
        } else {
            find_places();
            if (total > kMost * B) {  // nobody puts it together first: it is read where it lies
                if (tid == 0) st->redo |= kRedoList;
                const u32 mine = tid < G ? (c + entry.kPiece - 1u) / entry.kPiece : 0u, upto = block_scan<B>(mine, sm.wsum);
                if (tid != G) piece[tid] = tid < G ? upto - mine : ~0u;
                if (tid == B - 1) piece[G] = upto;
                __syncthreads();
                order_shared<DT, B>(P, row, rs, sm, shared, entry, total, 0u, 0u, 1u);
                return;
            }
            // 16 entries per thread are cut down
            const bool held = !few && __builtin_amdgcn_readfirstlane(__syncthreads_or(c > slots ? 1 : 0)) == 0;  // (every segment has places enough; else entries look for themselves)
#pragma unroll
            for (u32 j = 0; j < kMost; ++j) {
                const u32 i = tid + j * (u32)B, a = i >> log, l = i & (slots - 1u);
                if (!held) e[j] = i < total ? entry(i) : ~0ull;
                else if (i >= places || l >= segs[a + 1u] - segs[a]) e[j] = ~0ull;
            }
            bool crowd;
            n = __builtin_amdgcn_readfirstlane(keep_best<B>(e, total, rs.k, sm, &crowd));
            if ((crowd || total > L.most) && tid == 0) st->redo |= kRedoList;
        }
    } else if (__builtin_expect(over, 0)) {
        find_places();
        for (u32 i = tid; i < total; i += B) sm.buf[i] = entry(i);
    } else {
#pragma unroll
        for (u32 j = 0; j < kMost; ++j) {
            const u32 i = tid + j * (u32)B, a = i >> log, l = i & (slots - 1u);
            if (i < places && l < segs[a + 1u] - segs[a]) sm.buf[segs[a] + l] = e[j];
        }
        // (k_list_sweep's 512 segments: one of them has a little more than its places in every other row.  k_list_stream's have not, and 0.15 us to lose here.)
        if (few && ballot64(c > slots) != 0u) {
            const u32 at = list_segment<DT>(rs, tid, G, unit);
            for (u32 l = slots; l < c; ++l) sm.buf[segs[tid] + l] = from[at + l];
        }
    }
    order_list<DT, B>(P, row, rs, sm, n);
}

// k_list_part's lists: L.G of at most L.seg_stride entries, 8 B in all at most (so fewer than B lists).
// Bound by latency: the lists' lengths and the row's record come in one trip to memory.  In two, one row of 2^18 fp32 keys, k = 3 and 32, took 12.3 and 14.2 us;
// so 12.0 and 13.6.  An entry's list is guessed from their average length (found by halving, k = 48, 16.2 / 14.8).  Places and lengths read together, and
// the entries then put together in LDS, took 0.6 us more.
template <int DT, int B>
__global__ void __launch_bounds__(B) k_part_finish(Params P, ListPlan L) {
    __shared__ OrderShared<B> sm;
    __shared__ u32 segs[B + 1];
    const u32 tid = threadIdx.x, G = (u32)L.G;
    const int row = (int)blockIdx.x;
    const u32 c = tid < G ? list_part<u32>(P, row, L.seg_off)[tid] : 0u;
    if (list_row(P, row)->mode == kListSkip) return;
    const RowShape rs = row_shape_scalar<DT>(P, row);
    const u32 incl = block_scan<B>(c, sm.wsum);
    segs[tid] = incl - c;
    if (tid == B - 1) segs[B] = incl;
    __syncthreads();
    const u32 total = segs[B];
    const u64* from = list_array(P, 1u, row);
    const float per = (float)G / (float)total;
    auto entry = [&](u32 i) __attribute__((always_inline)) {  // (the lists are about equally long)
        u32 a = (u32)((float)i * per);
        a = a < G ? a : G - 1u;
        while (segs[a] > i) --a;
        while (segs[a + 1u] <= i) ++a;
        return from[a * L.seg_stride + (i - segs[a])];
    };
    rtopk_row_trace* st = row_state(P, row);
    if (tid == 0) list_record(st, rs, total, 5u);
    if (total < rs.k || total > 8u * B) {  // never expected: every stretch lists its k best
        if (tid == 0) st->error |= 4u;
        return;
    }
    // (a list that fewer waves can put in order is left to them: barriers)
    if (B > 256 && total <= 8u * 256u) {
        if (tid >= 256u) return;
        order_in_lds<DT, 256>(P, row, rs, *(OrderShared<256>*)&sm, total, 0u, entry);
    } else {
        order_in_lds<DT, B>(P, row, rs, sm, total, 0u, entry);
    }
}

// ------------------------------------------------------------------------------------------------
// one workgroup per row
// ------------------------------------------------------------------------------------------------

// B lanes hold a stretch of a row, NV vectors of 16 bytes each from vector p0 on (a multiple of B * NV; `last`: it is the
// row's last stretch): read once, in one go, and everything else works on registers.  Leaves a list in sm.ord.buf that
// contains the best min(k, size) elements of the stretch, and returns its length, at most `limit` (at least k + k / 16 + 2, or
// the stretch's size).  after_load() runs while the loads are under way.  Ends with a barrier.
// The bound needs no sample: the best element of every lane is known, and the k-th best of those is a number that at least
// k elements reach -- hardly more than k while k is small against B (k = B / 2: 1.4 k on independent draws).  For
// larger k the maxima of vectors take the place of the lanes'.
// A list that comes out too long (crowded keys) is bounded again by the exact k-th key, and if it is still too long, equal
// elements are added in the order of their positions until there are k.
template <int B>
struct HeldShared {
    static constexpr int OB = B < 256 ? B : 256;  // threads that order a short list
    union { OrderShared<B> ord; OrderShared<OB> few; RankShared rank; };  // (both lists at the same place)
    u32 part[2 * (B / 64)], run;
};
// The entry that hold_and_list left at place i of the list.  Where it left places in the row (*places), the elements are fetched from the caches here, all at once (to select one of 64
// registers by a number takes longer).  Fetched by the lane that noted them, one after the other, two or three trips: us, then / so, one fp32 row of 2^16, k = 32, 11.95 / 11.75, 16 rows of 2^17 bf16
// keys, k = 50, 14.2 / 14.0, 300 of 30011 fp16 keys, k = 100, 15.25 / 14.9, 512 of 2^14 bf16 keys, k = 628, 20.65 / 19.95.
template <int DT>
__device__ __forceinline__ u64 held_entry(const Params& P, const RowShape& rs, const u64* buf, u32 i, bool places) {
    const u64 v = buf[i];
    if (!places) return v;
    return list_entry<DT>(P).of(KeyOf<DT>::key(load_value<DT>(rs.x, (u32)v)) ^ P.dirmask, (u32)v);
}
template <int DT, int B, int NV, class AfterLoad>
__device__ __forceinline__ u32 hold_and_list(const Params& P, const RowShape& rs, u32 p0, bool last, u32 limit, HeldShared<B>& sm,
                                             bool* places, AfterLoad&& after_load) {
    constexpr int kGroups = NV / 4;  // the stretch as tiles of four vectors per lane
    typedef KeySource<DT, B, 4, false> Source;
    constexpr u32 E = Source::E;
    const u32 tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    Source src;
    src.init(rs);
    const bool largest = P.dirmask == 0;
    // Whole vectors of the row are held; lanes without one hold the worst number there is.  The few elements before the
    // first and after the last whole vector (a row may begin and end anywhere) go to the list unseen.
    const u32 worst = (DT == RTOPK_F32 ? 0x7f800000u : DT == RTOPK_F16 ? 0x7c007c00u : 0x7f807f80u) |
                      (largest ? (DT == RTOPK_F32 ? 0x80000000u : 0x80008000u) : 0u);
    typename Source::Tile t[kGroups];
    const u32 nvec = (u32)src.nvec, v0 = src.lead != 0u ? 1u : 0u, v1 = (u32)(((u64)src.lead + rs.n) / E);
    static_for<0, kGroups>([&](auto gc) __attribute__((always_inline)) {
        constexpr int g = decltype(gc)::value;
        static_for<0, 4>([&](auto uc) __attribute__((always_inline)) {
            constexpr int u = decltype(uc)::value;
            const u32 v = p0 + (u32)(4 * g + u) * B + tid;
            t[g].r[u] = make_uint4(worst, worst, worst, worst);
            if (v >= v0 && v < v1) t[g].r[u] = load16<false>(src.abase + v);
        });
    });
    // (the elements before the first whole vector belong to the first stretch, those after the last one to the last)
    const u32 before = src.lead != 0u ? (E - src.lead < rs.n ? E - src.lead : rs.n) : 0u;
    const u32 behind = rs.n - before - (v1 > v0 ? (v1 - v0) * E : 0u);
    const u32 head = p0 == 0u ? before : 0u, odd = head + (last ? behind : 0u);
    after_load();
    // (nothing computed from the elements in one phase is worth keeping for the next: unpacked, they would take twice the
    // registers)
    auto forget = [&]() __attribute__((always_inline)) {
        static_for<0, kGroups>([&](auto gc) __attribute__((always_inline)) {
            constexpr int g = decltype(gc)::value;
            static_for<0, 4>([&](auto uc) __attribute__((always_inline)) {
                uint4& q = t[g].r[decltype(uc)::value];
                asm volatile("" : "+v"(q.x), "+v"(q.y), "+v"(q.z), "+v"(q.w));
            });
        });
    };
    auto better = [&](float a, float b) __attribute__((always_inline)) { return largest ? __builtin_fmaxf(a, b) : __builtin_fminf(a, b); };
    auto best_of_vector = [&](const typename Source::Tile& tile, auto uc) __attribute__((always_inline)) {
        constexpr int u = decltype(uc)::value;
        float m = src.template value<SRC_KEY>(tile, u * (int)E, 0.0f);
        static_for<1, (int)E>([&](auto jc) __attribute__((always_inline)) {
            m = better(m, src.template value<SRC_KEY>(tile, u * (int)E + decltype(jc)::value, 0.0f));
        });
        return m;
    };
    // the order of numbers as 32-bit keys (those of fp32, for every type)
    auto key_of_number = [&](float x) __attribute__((always_inline)) { return KeyOf<RTOPK_F32>::key(__float_as_uint(x)) ^ (largest ? 0u : 0xffffffffu); };
    u32 T, top;
    bool exact;
    {
        float m = best_of_vector(t[0], std::integral_constant<int, 0>{});
        static_for<0, kGroups>([&](auto gc) __attribute__((always_inline)) {
            constexpr int g = decltype(gc)::value;
            static_for<0, 4>([&](auto uc) __attribute__((always_inline)) {
                m = better(m, best_of_vector(t[g], uc));
                __builtin_amdgcn_sched_barrier(0);
            });
        });
        forget();
        const u32 lmax = key_of_number(m);
        top = wave_reduce(lmax, MaxOf());
        u32 low = wave_reduce(lmax, MinOf());
        if (lane == 63u) {
            sm.part[2 * wave] = top;
            sm.part[2 * wave + 1] = low;
        }
        __syncthreads();
        top = sm.part[0];
        low = sm.part[1];
#pragma unroll
        for (int w = 1; w < B / 64; ++w) {
            top = top > sm.part[2 * w] ? top : sm.part[2 * w];
            low = low < sm.part[2 * w + 1] ? low : sm.part[2 * w + 1];
        }
        __syncthreads();
        if (rs.k <= (u32)B / 2u) {
            sm.rank.hist[tid] = lmax;
            T = rank_by_one_wave<B>(rs.k, low, top, sm.rank.hist, sm.rank.selv, &exact);
        } else if (NV < 16 && rs.k <= (u32)(B * NV) / 2u) {  // (with 16 vectors the registers do not allow it)
            T = sample_rank<B>([&](auto&& f) __attribute__((always_inline)) {
                static_for<0, kGroups>([&](auto gc) __attribute__((always_inline)) {
                    constexpr int g = decltype(gc)::value;
                    static_for<0, 4>([&](auto uc) __attribute__((always_inline)) {
                        f(key_of_number(best_of_vector(t[g], uc)));
                        __builtin_amdgcn_sched_barrier(0);
                    });
                });
            }, rs.k, 0u, top, sm.rank, &exact);
        } else {
            T = 0;
        }
    }
    forget();
    // masks of what is not worse than the number T stands for; it has to be better than what lies outside the row
    u32 m[kGroups], mine = 0;
    const float x = __uint_as_float(largest ? ((T & 0x80000000u) ? T ^ 0x80000000u : ~T) : ((T & 0x80000000u) ? T : T ^ 0x7fffffffu));
    const bool bounded = T != 0u && (largest ? x > -__builtin_inff() : x < __builtin_inff());
    static_for<0, kGroups>([&](auto gc) __attribute__((always_inline)) {
        constexpr int g = decltype(gc)::value;
        u32 worse = 0;
        static_for<0, Source::kSlots>([&](auto sc) __attribute__((always_inline)) {
            const float v = src.template value<SRC_KEY>(t[g], decltype(sc)::value, 0.0f);
            worse = largest ? shift_in_below(worse, v, x) : shift_in_not_up_to(worse, v, x);  // (NaNs are the best, or the worst)
        });
        __builtin_amdgcn_sched_barrier(0);
        m[g] = worse ^ (0xffffffffu >> (32 - Source::kSlots));
        mine += (u32)__builtin_popcount(m[g]);
    });
    u32 pos = odd + block_scan<B>(mine, sm.part) - mine;  // this lane's place in the list
    u32 listed = odd;
#pragma unroll
    for (int w = 0; w < B / 64; ++w) listed += sm.part[w];
    const ListEntry ent = list_entry<DT>(P);
    __syncthreads();  // (the counting arrays are done with)
    if (listed <= limit && bounded) {
        if (tid < odd) sm.ord.buf[tid] = tid < head ? tid : rs.n - odd + tid;
        for (;;) {
            u32 left = 0, group = 0;
            static_for<0, kGroups>([&](auto gc) __attribute__((always_inline)) {
                constexpr int g = kGroups - 1 - decltype(gc)::value;
                if (m[g] != 0u) { left = m[g]; group = (u32)g; }
            });
            if (ballot64(left != 0u) == 0) break;
            const u32 bit = 31u - (u32)__builtin_clz(left | 1u), s = (u32)Source::kSlots - 1u - bit;
            static_for<0, kGroups>([&](auto gc) __attribute__((always_inline)) {
                constexpr int g = decltype(gc)::value;
                if (left != 0u && group == (u32)g) m[g] ^= 1u << bit;
            });
            if (left != 0u) sm.ord.buf[pos++] = element_index(src, p0 / (4u * B) + group, s);
        }
        __syncthreads();
        *places = true;
        return listed;
    }
    *places = false;
    // Crowded, or k close to the stretch's size: the k-th key itself, of all elements (which are read again: the caches have
    // them, and the registers stay free of what this rare way needs).
    const u32 pend = last || p0 + (u32)(B * NV) > nvec ? nvec : p0 + (u32)(B * NV);
    auto all = [&](auto&& f) __attribute__((always_inline)) {
#pragma unroll 1
        for (u32 v = p0 + tid; v < pend; v += B) {
            uint4 q = load16<false>(src.abase + v);
            keys_of_vector<DT>(q, P.dirmask);
#pragma unroll
            for (u32 j = 0; j < E; ++j) {
                const u32 idx = v * E + j - src.lead;
                if (idx < rs.n) f(key_in_vector<DT>(q, (int)j), idx);
            }
        }
    };
    const u32 from = p0 == 0u ? 0u : p0 * E - src.lead, to = pend * E - src.lead < rs.n ? pend * E - src.lead : rs.n;
    const u32 size = pend > p0 ? to - from : 0u;
    u32 Tk = 0;
    if (size > limit) {  // (a stretch that the list holds whole needs no bound)
        // It lies between T and the best number (crowds: often the same, and there is nothing left to do), or among the NaNs, which
        // were passed over.  Elements' keys; a fp16 number near T is rounded, hence one key lower.  (Elements outside
        // whole vectors are no part of those: they count as better where they are.)
        constexpr u32 ksh = DT == RTOPK_F32 ? 0u : 16u;
        auto key_of = [&](u32 k32) __attribute__((always_inline)) {
            if constexpr (DT != RTOPK_F16) {
                return k32 >> ksh;
            } else {
                const u32 o = largest ? k32 : ~k32;
                const float f = __uint_as_float((o & 0x80000000u) ? o ^ 0x80000000u : ~o);
                return (KeyOf<DT>::key((u32)__builtin_bit_cast(uint16_t, (_Float16)f)) ^ P.dirmask) >> ksh;
            }
        };
        const u32 last_key = 0xffffffffu >> ksh;
        u32 lo = bounded ? key_of(T) : 0u, hi = key_of(top), rank = rs.k, above = 0;
        if (DT == RTOPK_F16 && lo != 0u) --lo;
        all([&](u32 key, u32) __attribute__((always_inline)) { above += (key >> ksh) > hi ? 1u : 0u; });
        above = wave_inclusive_scan(above);
        __syncthreads();
        if (lane == 63u) sm.part[wave] = above;
        __syncthreads();
        above = sum_of_waves<B>(sm.part, 1);
        if (above >= rank) {
            lo = hi + 1u;
            hi = last_key;
        } else {
            rank -= above;
        }
        if (lo >= hi) {
            Tk = hi;
            exact = true;
        } else {
            Tk = sample_rank<B>([&](auto&& f) __attribute__((always_inline)) { all([&](u32 key, u32) __attribute__((always_inline)) { f(key >> ksh); }); },
                                rank, lo, hi, sm.rank, &exact);
        }
        Tk <<= ksh;
    }
    bool tied = false;
    for (;;) {  // what is not below it; if that is too much, what is above it
        if (tid == 0) sm.run = 0;
        __syncthreads();
        all([&](u32 key, u32 idx) __attribute__((always_inline)) {
            if (key > Tk || (key == Tk && !tied)) {
                const u32 at = atomicAdd(&sm.run, 1u);
                if (at < limit) sm.ord.buf[at] = ent.of(key, idx);
            }
        });
        __syncthreads();
        listed = sm.run;
        if (listed <= limit || tied) break;
        tied = true;
        __syncthreads();
    }
    // equal elements, a vector per thread at a time: thread order is position order
    for (u32 b = p0; tied && listed < rs.k && b < pend; b += B) {
        const u32 v = b + tid;
        u32 hit = 0;
        if (v < pend) {
            uint4 q = load16<false>(src.abase + v);
            keys_of_vector<DT>(q, P.dirmask);
#pragma unroll
            for (u32 j = 0; j < E; ++j) hit |= (v * E + j - src.lead < rs.n && key_in_vector<DT>(q, (int)j) == Tk ? 1u : 0u) << j;
        }
        const u32 n = (u32)__builtin_popcount(hit);
        u32 at = listed + block_scan<B>(n, sm.part) - n;
        for (; hit != 0u && at < rs.k; hit &= hit - 1u, ++at) sm.ord.buf[at] = ent.of(Tk, v * E + (u32)__builtin_ctz(hit) - src.lead);
#pragma unroll
        for (int w = 0; w < B / 64; ++w) listed += sm.part[w];
        if (listed > rs.k) listed = rs.k;
        __syncthreads();
    }
    return listed;
}

// A row that one workgroup can hold: no sample, one launch, no row left over.
// Bound by latency: one trip to memory, then about ten phases with barriers (the first four waves alone put a short list
// in order: a barrier among 16 waves takes 1 us, among 4 waves 0.5).
template <int DT, int B, int NV>
__global__ void __launch_bounds__(B, 4) k_list_held(Params P, ListPlan L) {
    constexpr u32 kCap = 8 * B;
    constexpr int OB = HeldShared<B>::OB;
    __shared__ HeldShared<B> sm;
    const int row = blockIdx.x;
    const u32 tid = threadIdx.x;
    const RowShape rs = row_shape_scalar<DT>(P, row);
    rtopk_row_trace* st = row_state(P, row);
    if (rs.k == 0) {
        init_row<DT>(P, row, st, rs);
        return;
    }
    bool places;
    const u32 listed = hold_and_list<DT, B, NV>(P, rs, 0u, true, kCap, sm, &places, [&]() __attribute__((always_inline)) { init_row<DT>(P, row, st, rs); });
    if (tid == 0) list_record(st, rs, listed, 6u);
    if (listed > kCap) {  // never expected: the k-th key bounds the list
        if (tid == 0) st->error |= 4u;
    } else if (listed <= 8u * OB) {
        if (tid >= (u32)OB) return;  // (a barrier waits for the waves that are left)
        order_in_lds<DT, OB>(P, row, rs, sm.few, listed, 0u, [&](u32 i) __attribute__((always_inline)) { return held_entry<DT>(P, rs, sm.few.buf, i, places); });
    } else {
        order_in_lds<DT, B>(P, row, rs, sm.ord, listed, 0u, [&](u32 i) __attribute__((always_inline)) { return held_entry<DT>(P, rs, sm.ord.buf, i, places); });
    }
}

// Few rows, small k: a row's stretches of 32 KB are held by a workgroup each, which list their best k; k_part_finish puts a
// row's L.G lists of at most L.seg_stride entries in order.  Two launches, no sample, no row left over.
constexpr int kPartBlock = kListPartBlock, kPartVecs = kListPartVecs;
template <int DT>
__global__ void __launch_bounds__(kPartBlock, 4) k_list_part(Params P, ListPlan L) {
    constexpr int B = kPartBlock;
    __shared__ HeldShared<B> sm;
    const u32 G = (u32)L.G, tid = threadIdx.x;
    const int row = (int)(blockIdx.x / G);
    const u32 g = blockIdx.x % G;
    const RowShape rs = row_shape_scalar<DT>(P, row);
    rtopk_row_trace* st = row_state(P, row);
    KeySource<DT, B, 4, false> src;
    src.init(rs);
    constexpr u32 kHeld = (u32)B * (u32)kPartVecs;
    const u32 p0 = g * kHeld, nvec = (u32)src.nvec;
    u32 listed = 0;
    auto first = [&]() __attribute__((always_inline)) {
        if (g == 0u) {
            init_row<DT>(P, row, st, rs);
            if (tid == 0) list_row_out(P, row)->mode = rs.k == 0u ? kListSkip : kListPlain;
        }
    };
    if (rs.k == 0u || p0 >= nvec) {
        first();
    } else {
        bool places;
        listed = hold_and_list<DT, B, kPartVecs>(P, rs, p0, p0 + kHeld >= nvec, L.seg_stride, sm, &places, first);
        u64* seg = list_array(P, 1u, row) + (size_t)g * L.seg_stride;
        for (u32 i = tid; i < listed && i < L.seg_stride; i += B) seg[i] = held_entry<DT>(P, rs, sm.ord.buf, i, places);
    }
    if (tid == 0) list_part<u32>(P, row, L.seg_off)[g] = listed < L.seg_stride ? listed : L.seg_stride;
}

// (Registers: six waves to a SIMD where a workgroup has eight, which what is normally not there to be done would else make four: 1024 rows of 2^17 bf16 keys, k = 1024, 68.8 us / 63.9.
// Workgroups of four waves are better four to a compute unit than unevenly more of them: k = 50, six waves 52.4 us, four 49.4.  Ties are summed up, and a row selected anew, where they are found to be too few:
// with that known before the list is ordered, as elsewhere, and both ways of ordering behind it, k = 50 49.2 / 49.8 and k = 1024 62.7 / 63.3, 1000 rows of 50257, k = 100, 31.7 / 32.6.)
// Bound, sweep and order in one kernel: the list is gathered in LDS (what does not fit there goes to the list array).
// For rows so short, or so many, that sharing one out gains nothing.  Several of these workgroups share a compute unit, so that one
// row's trip from memory overlaps the others' ranking.
template <int DT, int B, int V, bool NT>
__global__ void __launch_bounds__(B, B == 512 ? 6 : 4) k_list_row(Params P, ListPlan L) {
    constexpr int OB = B < 256 ? B : 256;  // threads that order a short list (see k_list_held)
    __shared__ union { OrderShared<B> ord; OrderShared<OB> few; RankShared rank; } sm;
    __shared__ OrderParts<B> shared;
    __shared__ ListRow lr;
    __shared__ u32 red[3 * (B / 64)], te[kListRowTiles], run;
    constexpr u32 kCap = 8 * B;
    typedef KeySource<DT, B, 4, NT> Source;
    const int row = blockIdx.x;
    const u32 tid = threadIdx.x, lane = lane_id();
    const RowShape rs = row_shape_scalar<DT>(P, row);
    rtopk_row_trace* st = row_state(P, row);
    Source src;
    src.init(rs);
    bound_of_row<DT, B, V, false, 8>(P, L, row, rs, st, &lr, te, src.ntiles(), kCap, sm.rank, nullptr, red, true, [] {});
    if (tid == 0) run = 0;
    __syncthreads();
    if (lr.mode == kListSkip) return;
    const ListRow b = list_row_scalar(&lr);
    const ListEntry ent = list_entry<DT>(P);
    u64* list = list_array(P, 1u, row);
    (void)sweep_row<DT>(src, 0u, 1u, b, te, P.dirmask, [&](const typename Source::Tile& cur, u32 m) __attribute__((always_inline)) {
        for (;;) {
            const u64 have = ballot64(m != 0u);
            if (have == 0) break;
            u32 base = 0;
            if (lane == 0) base = atomicAdd(&run, (u32)__popcll(have));
            base = __builtin_amdgcn_readfirstlane(base);
            if (m != 0u) {
                const u32 bit = 31u - (u32)__builtin_clz(m), s = (u32)Source::kSlots - 1u - bit;
                m ^= 1u << bit;
                const u32 pos = base + mbcnt64(have);
                const u64 e = ent.of(KeyOf<DT>::key(pick<Source>(cur, s)) ^ P.dirmask, element_index(src, cur.tile, s));
                if (pos < kCap) sm.ord.buf[pos] = e;
                else list[pos] = e;
            }
        }
    });
    __syncthreads();
    const u32 total = run;
    if (b.mode == kListPlain && total < rs.k) {
        const u32 n = redo_row<DT, B, false>(P, L, row, rs, st, 8u, sm.ord, sm.rank, &run);
        if (n != 0u) order_in_lds<DT, B>(P, row, rs, sm.ord, n, 0u, [&](u32 i) __attribute__((always_inline)) { return sm.ord.buf[i]; });
        return;
    }
    if (tid == 0) list_record(st, rs, total, 6u);
    if (total > kCap) {
        for (u32 i = tid; i < kCap; i += B) list[i] = sm.ord.buf[i];
        if (tid == 0) st->redo |= kRedoList;
        order_shared<DT, B>(P, row, rs, sm.ord, shared, EntriesAt{list}, total, 0u, 0u, 1u);
    } else if (total != 0u && total <= 8u * OB && b.mode != kListTied) {
        if (tid >= (u32)OB) return;  // (a barrier waits for the waves that are left)
        order_in_lds<DT, OB>(P, row, rs, sm.few, total, 0u, [&](u32 i) __attribute__((always_inline)) { return sm.few.buf[i]; });
    } else if (total != 0u) {
        order_in_lds<DT, B, false, (B > 512)>(P, row, rs, sm.ord, total, 0u, [&](u32 i) __attribute__((always_inline)) { return sm.ord.buf[i]; });
    }
    if (b.mode == kListTied && total < rs.k) {
        __syncthreads();
        if (!ties_of_row<DT, B, Source>(P, TileCounts{te}, row, rs, total, b.T, 0u, 1u, sm.ord.hist, sm.ord.wsum)) {
            __syncthreads();
            const u32 n = redo_row<DT, B, false>(P, L, row, rs, st, 8u, sm.ord, sm.rank, &run);
            if (n != 0u) order_in_lds<DT, B>(P, row, rs, sm.ord, n, 0u, [&](u32 i) __attribute__((always_inline)) { return sm.ord.buf[i]; });
        }
    }
}

// ------------------------------------------------------------------------------------------------
// long lists
// ------------------------------------------------------------------------------------------------

constexpr u32 kBucketRoom = 8 * kListBucketBlock;  // entries of a bucket that one workgroup puts in order

// The elements equal to T that the row's workgroups counted, into *sum (which has been cleared before a barrier).
__device__ __forceinline__ void add_ties(u32 mode, u32 mine, u32* sum) {
    if (mode != kListTied) return;
    mine = wave_inclusive_scan(mine);
    if (lane_id() == 63u && mine != 0u) atomicAdd(sum, mine);
}

// Thread t's bins of a list's histogram, the 4 t-th best and the three below it, added up over its copies.
__device__ __forceinline__ void list_counts(const Params& P, const ListPlan& L, int row, u32 (&c)[4]) {
    static_assert(kListBins == 4 * kLongBlock, "four to a thread");
    const uint4* gh = list_part<uint4>(P, row, L.hist_off) + (kListBins / 4u - 1u - threadIdx.x);
    uint4 a = gh[0];
    if (L.hists == 4u) {
        const uint4 x = gh[kListBins / 4u], y = gh[2u * (kListBins / 4u)], z = gh[3u * (kListBins / 4u)];
        a = make_uint4(a.x + x.x + y.x + z.x, a.y + x.y + y.y + z.y, a.z + x.z + y.z + z.z, a.w + x.w + y.w + z.w);
    }
    c[0] = a.w;
    c[1] = a.z;
    c[2] = a.y;
    c[3] = a.x;
}

// Workgroup w moves segment w into buckets.  A bin's rank is the number of entries in better bins; a bucket is the run of
// bins whose ranks share rank >> L.bucket_shift, its place in the array its first bin's rank.  A bin that ends beyond the ranks of the next bucket, which is
// then left without any, is that one alone: else its bucket, with what begins before it, would be longer than one workgroup puts in order.  Bins that begin at rank k or
// beyond are dropped.  One atomic per bucket reserves all of a workgroup's places in it; what the registers do not hold
// of a segment is read twice.  Those atomics are waited for, and the ones to one counter are made one after the other, 11 ns each: of a single row's, every other workgroup takes its
// places from the bucket's end, with a counter of its own.  A single row has one more workgroup, without a segment, which writes down where the buckets begin while the others move
// theirs (each bucket's size from its last bin: searched for, the next bucket that has any bins is far where there are few).  Several rows' would share compute units with others: eight rows of
// 2^19 fp32 keys, k = 52428, 42.0 us, with them 42.4 to 43.4.  us, one counter and workgroup 0 with records and search / so: one fp32 row of 2^28
// keys, k = 2^20, 218 / 216; of 2^22 + 3 fp16 keys, k = 2^20, 59.2 / 58.2; nine in ten equal, 8.3 million fp16 keys, k = n / 8, 120 / 85, 2^26 fp32 keys, k = 2^16, 86.0 / 84.5.
template <int DT>
__global__ void __launch_bounds__(kLongBlock) k_list_scatter(Params P, ListPlan L) {
    constexpr int B = kLongBlock, kPer = kListBins / B;
    __shared__ u32 bucket[kListBins];        // of every bin, or ~0
    __shared__ u32 place[kListMaxBuckets];   // of every bucket: this workgroup's entries, then their next place
    __shared__ u64 split[kListSplits + 1];
    __shared__ u32 wsum[B / 64];
    __shared__ u32 s_end, s_total, s_equal, s_big;
    const u32 G = (u32)L.G, tid = threadIdx.x;
    const bool alone = P.batch == 1;  // (of several rows: workgroup 0)
    const int row = alone ? 0 : (int)(blockIdx.x / G);
    const u32 wg = alone ? blockIdx.x : blockIdx.x % G;
    const bool records = wg == (alone ? G : 0u);
    const ListRow* lr = list_row(P, row);
    const u32 mode = lr->mode;
    if (mode == kListSkip) return;
    const RowShape rs = row_shape_scalar<DT>(P, row);
    rtopk_row_trace* st = row_state(P, row);
    const u64 lo = lr->lo;
    const u32 sh = lr->sh, by_split = __builtin_amdgcn_readfirstlane(lr->split);
    if (by_split != 0u && tid <= kListSplits) split[tid] = list_part<u64>(P, row, L.split_off)[tid];
    const u64* from = list_array(P, 1u, row) + list_segment<DT>(rs, wg, G, long_unit(L));
    const uint2* segs = list_part<uint2>(P, row, L.seg_off);
    const u32 mine = wg == G ? 0u : segs[wg].x;
    const u32 equal = mode == kListTied && tid < G ? segs[tid].y : 0u;  // (G is at most 256)
    constexpr int kHeld = 8;
    u64 held[kHeld];
#pragma unroll
    for (int i = 0; i < kHeld; ++i) held[i] = tid + (u32)i * B < mine ? from[tid + (u32)i * B] : 0ull;
    const u32 bs = L.bucket_shift, nb = L.nb;
    u32 c[kPer], s = 0, rank[kPer];
    list_counts(P, L, row, c);
#pragma unroll
    for (int i = 0; i < kPer; ++i) s += c[i];
    for (u32 j = tid; j < nb; j += B) place[j] = 0;
    if (tid == 0) s_end = s_equal = s_big = 0;
    const u32 incl = block_scan<B>(s, wsum);
    {
        u32 r = incl - s;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const u32 j = (r >> bs) + 1u;
            bucket[kListBins - 1u - (tid * kPer + i)] = r >= rs.k ? 0xffffffffu : j < nb && r + c[i] > ((j + 1u) << bs) ? j : j - 1u;
            rank[i] = r;
            if (r < rs.k && r + c[i] >= rs.k) s_end = r + c[i];
            r += c[i];
        }
        if (tid == B - 1) s_total = r;
    }
    add_ties(mode, equal, &s_equal);
    // f(bucket, rank) for this thread's bins that begin one, or end one
    auto first_bins = [&](auto&& f) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const u32 q = tid * kPer + i, b = bucket[kListBins - 1u - q];
            if (b != 0xffffffffu && (q == 0u || b != bucket[kListBins - q])) f(b, rank[i]);
        }
    };
    auto last_bins = [&](auto&& f) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const u32 q = tid * kPer + i, b = bucket[kListBins - 1u - q];
            if (b != 0xffffffffu && (q == kListBins - 1u || b != bucket[kListBins - 2u - q])) f(b, rank[i] + c[i]);
        }
    };
    __syncthreads();
    const u32 total = s_total;
    const bool few = total < rs.k;
    const u32 end = few ? total : s_end;
    const bool few_in_all = few && (u64)total + s_equal < (u64)rs.k;
    const bool drop = few_in_all || end > (u32)((P.n + 1) / 2);  // (the buckets have half a candidate array)
    if (drop) {
        if (records && tid == 0) *list_done(P, row) = ListDone{total, few_in_all ? 8u : 5u, 0u};
        return;
    }
    if (records) {
        if (tid == 0) list_record(st, rs, total, 5u);
        // the buckets' first ranks and sizes
        u32* first = list_part<u32>(P, row, L.first_off);
        for (u32 j = tid; j < nb; j += B) place[j] = 0xffffffffu;
        __syncthreads();
        first_bins([&](u32 b, u32 r) __attribute__((always_inline)) { place[b] = r; });
        __syncthreads();
        last_bins([&](u32 b, u32 r) __attribute__((always_inline)) {
            const u32 size = r - place[b];
            first[2u * b + 1u] = size;
            if (size > kBucketRoom) s_big = 1u;
        });
        for (u32 j = tid; j < nb; j += B) first[2u * j] = place[j];  // (~0: no bin begins it, and it has no size)
        __syncthreads();
        if (tid == 0) *list_done(P, row) = ListDone{total, 0u, s_big};
        if (alone) return;
        for (u32 j = tid; j < nb; j += B) place[j] = 0;
        __syncthreads();
    }
    auto bucket_of = [&](u64 e) __attribute__((always_inline)) { return bucket[by_split != 0u ? list_bin_split(e, split) : list_bin(e, lo, sh)]; };
    // (what the registers hold of the segment is on its way before the ranks are known)
    u32 bk[kHeld];
#pragma unroll
    for (int i = 0; i < kHeld; ++i) {
        bk[i] = 0xffffffffu;
        if (tid + (u32)i * B < mine) bk[i] = bucket_of(held[i]);
        if (bk[i] != 0xffffffffu) atomicAdd(&place[bk[i]], 1u);
    }
    for (u32 i = tid + kHeld * B; i < mine; i += B) {
        const u32 b = bucket_of(from[i]);
        if (b != 0xffffffffu) atomicAdd(&place[b], 1u);
    }
    __syncthreads();
    const u32 back = alone ? wg & 1u : 0u;  // (several rows' have few workgroups each)
    u32* cursor = list_part<u32>(P, row, L.cursor_off) + back * list_cursors(nb);
    // a bucket's own beginning is added by the bin that begins it, its end by the one that ends it
    for (u32 j = tid; j < nb; j += B) {
        const u32 n = place[j];
        if (n != 0) {
            const u32 before = atomicAdd(&cursor[j], n);
            place[j] = back != 0u ? 0u - before - n : before;
        }
    }
    __syncthreads();
    if (back != 0u) last_bins([&](u32 b, u32 r) __attribute__((always_inline)) { place[b] += r; });
    else first_bins([&](u32 b, u32 r) __attribute__((always_inline)) { place[b] += r; });
    __syncthreads();
    u64* dst = list_array(P, 0u, row);
#pragma unroll
    for (int i = 0; i < kHeld; ++i)
        if (bk[i] != 0xffffffffu) dst[atomicAdd(&place[bk[i]], 1u)] = held[i];
    for (u32 i = tid + kHeld * B; i < mine; i += B) {
        const u64 e = from[i];
        const u32 b = bucket_of(e);
        if (b != 0xffffffffu) dst[atomicAdd(&place[b], 1u)] = e;
    }
}

// Unsorted output.  Workgroup w writes segment w: entries of better bins than the one rank k - 1 lies in go straight to the output, in whatever order they
// are in, those of that bin to the row's only bucket, which k_list_buckets takes the missing ones from.  One atomic per workgroup reserves its places.
// (2^26 fp32 keys, k = n / 100, through the buckets, every one of which is then put in order: 14.1 + 10.0 us; so 8.9 + 5.4, and what the caller
// does with positions that lie near one another is faster, too.)
template <int DT>
__global__ void __launch_bounds__(kLongBlock) k_list_emit(Params P, ListPlan L) {
    constexpr int B = kLongBlock, kPer = kListBins / B, kHeld = 8;
    __shared__ u64 split[kListSplits + 1], s_base;
    __shared__ u32 wsum[B / 64], counts[2 * (B / 64)], s_bin, s_rank, s_end, s_equal;
    const u32 G = (u32)L.G, tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const int row = (int)(blockIdx.x / G);
    const u32 wg = blockIdx.x % G;
    const ListRow* lr = list_row(P, row);
    const u32 mode = lr->mode;
    if (mode == kListSkip) return;
    const RowShape rs = row_shape_scalar<DT>(P, row);
    rtopk_row_trace* st = row_state(P, row);
    const u64 lo = lr->lo;
    const u32 sh = lr->sh, by_split = __builtin_amdgcn_readfirstlane(lr->split);
    if (by_split != 0u && tid <= kListSplits) split[tid] = list_part<u64>(P, row, L.split_off)[tid];
    const u64* from = list_array(P, 1u, row) + list_segment<DT>(rs, wg, G, (u32)kLongBlock * 4u);  // (no half tiles: the plan has unsorted lists of rows of 2^25 keys and more)
    const uint2* segs = list_part<uint2>(P, row, L.seg_off);
    const u32 mine = segs[wg].x;
    const u32 equal = mode == kListTied && tid < G ? segs[tid].y : 0u;  // (G is at most 256)
    u64 held[kHeld];
#pragma unroll
    for (int i = 0; i < kHeld; ++i) held[i] = tid + (u32)i * B < mine ? from[tid + (u32)i * B] : 0ull;
    u32 c[kPer], s = 0;
    list_counts(P, L, row, c);
#pragma unroll
    for (int i = 0; i < kPer; ++i) s += c[i];
    if (tid == 0) {
        s_bin = 0xffffffffu;
        s_equal = 0;
    }
    const u32 incl = block_scan<B>(s, wsum);
    {
        u32 r = incl - s;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            if (r < rs.k && r + c[i] >= rs.k) {
                s_bin = kListBins - 1u - (tid * kPer + i);
                s_rank = r;
                s_end = r + c[i];
            }
            r += c[i];
        }
        if (tid == B - 1) counts[0] = r;
    }
    add_ties(mode, equal, &s_equal);
    __syncthreads();
    const u32 total = counts[0], bin = s_bin;  // (fewer than k in all: 0xffffffff, and every entry is output)
    const bool few = bin == 0xffffffffu;
    const u32 rank = few ? total : s_rank, end = few ? total : s_end;
    const bool few_in_all = few && (u64)total + s_equal < (u64)rs.k;
    const bool drop = few_in_all || end > (u32)((P.n + 1) / 2);  // (the bucket has its place in half a candidate array)
    if (wg == 0 && tid == 0) {
        *list_done(P, row) = ListDone{total, drop ? (few_in_all ? 8u : 5u) : 0u, !few && end - rank > kBucketRoom ? 1u : 0u};
        u32* first = list_part<u32>(P, row, L.first_off);
        first[0] = few ? 0xffffffffu : rank;
        first[1] = end - rank;
        if (!drop) list_record(st, rs, total, 5u);
    }
    if (drop) return;
    __syncthreads();  // (everybody has read the total)
    // 0: not wanted; 1: of the bin; 2: output
    auto what = [&](u64 e) __attribute__((always_inline)) {
        const u32 b = by_split != 0u ? list_bin_split(e, split) : list_bin(e, lo, sh);
        return few || b > bin ? 2u : b == bin ? 1u : 0u;
    };
    u32 is[kHeld], out = 0, in = 0;  // (of the wave: counts)
#pragma unroll
    for (int i = 0; i < kHeld; ++i) {
        is[i] = tid + (u32)i * B < mine ? what(held[i]) : 0u;
        out += (u32)__popcll(ballot64(is[i] == 2u));
        in += (u32)__popcll(ballot64(is[i] == 1u));
    }
    for (u32 i0 = wave * 64u + kHeld * B; i0 < mine; i0 += B) {  // (what the registers do not hold is read twice)
        const u32 w = i0 + lane < mine ? what(from[i0 + lane]) : 0u;
        out += (u32)__popcll(ballot64(w == 2u));
        in += (u32)__popcll(ballot64(w == 1u));
    }
    if (lane == 0) { counts[2 * wave] = out; counts[2 * wave + 1] = in; }
    __syncthreads();
    const u32 so = wave_inclusive_scan(lane < (u32)(B / 64) ? counts[2 * (lane % (u32)(B / 64))] : 0u);
    const u32 si = wave_inclusive_scan(lane < (u32)(B / 64) ? counts[2 * (lane % (u32)(B / 64)) + 1] : 0u);
    if (tid == 0) {
        const u64 n = (u64)(u32)__builtin_amdgcn_readlane((int)si, 63) << 32 | (u32)__builtin_amdgcn_readlane((int)so, 63);
        s_base = n != 0u ? atomicAdd((unsigned long long*)list_part<u64>(P, row, L.cursor_off), (unsigned long long)n) : 0u;
    }
    __syncthreads();
    u32 at_out = (u32)s_base + (u32)__shfl((int)so, (int)wave, 64) - out, at_in = rank + (u32)(s_base >> 32) + (u32)__shfl((int)si, (int)wave, 64) - in;
    const ListEntry ent = list_entry<DT>(P);
    char* out_v = (char*)P.out_values + (size_t)row * (size_t)P.k * KeyOf<DT>::kBytes;
    long long* out_i = P.out_indices + (size_t)row * (size_t)P.k;
    u64* dst = list_array(P, 0u, row);
    auto put = [&](u64 e, u32 w) __attribute__((always_inline)) {
        const u64 o = ballot64(w == 2u), b = ballot64(w == 1u);
        if (w == 2u) {
            const u32 p = at_out + mbcnt64(o), idx = ent.idx(e);
            out_i[p] = (long long)idx;
            store_value<DT>(out_v, p, raw_of_key<DT>(ent.key(e), idx, rs, P.dirmask));
        }
        if (w == 1u) dst[at_in + mbcnt64(b)] = e;
        at_out += (u32)__popcll(o);
        at_in += (u32)__popcll(b);
    };
#pragma unroll
    for (int i = 0; i < kHeld; ++i) put(held[i], is[i]);
    for (u32 i0 = wave * 64u + kHeld * B; i0 < mine; i0 += B) {
        const u64 e = i0 + lane < mine ? from[i0 + lane] : 0ull;
        put(e, i0 + lane < mine ? what(e) : 0u);
    }
}

// Where bucket j of a row begins and how many entries it has; false if there is no such bucket, or nothing is wanted from it.
__device__ __forceinline__ bool bucket_range(const Params& P, const ListPlan& L, int row, const RowShape& rs, u32 j, u32* at, u32* count) {
    const uint2 f = list_part<uint2>(P, row, L.first_off)[j];
    *at = f.x;
    *count = f.y;
    return f.x != 0xffffffffu && f.x < rs.k && f.y != 0u;  // (empty bins alone may begin one)
}

// One workgroup per bucket (blocks [0, nb) of a row) puts its entries in order; the other L.ties blocks of the row are for
// the elements equal to T.  Buckets of too many entries are shared out among all of a row's workgroups, and the first has a row whose list was no use.
template <int DT>
__global__ void __launch_bounds__(kListBucketBlock, 6) k_list_buckets(Params P, ListPlan L) {
    constexpr int B = kListBucketBlock;
    __shared__ union { OrderShared<B> ord; RankShared rank; } lds;
    __shared__ OrderParts<B> shared;
    __shared__ u32 before[B], run;
    OrderShared<B>& sm = lds.ord;
    const u32 per = L.nb + (u32)L.ties, tid = threadIdx.x;
    const int row = __builtin_amdgcn_readfirstlane((int)(blockIdx.x / per));
    const u32 j = __builtin_amdgcn_readfirstlane(blockIdx.x % per);
    const ListRow* lr = list_row(P, row);
    const u32 mode = lr->mode;
    if (mode == kListSkip) return;
    const ListDone done = *list_done(P, row);
    const RowShape rs = row_shape_scalar<DT>(P, row);
    rtopk_row_trace* st = row_state(P, row);
    if (done.drop != 0u) {
        if (j != 0u) return;
        const u32 n = redo_row<DT, B, true>(P, L, row, rs, st, done.drop, sm, lds.rank, &run);
        if (n != 0u) order_entries<DT, B>(P, row, rs, sm, 0u, n, 1u, list_part<OrderRange>(P, row, L.stack_off));
        return;
    }
    u32 at = 0, count = 0;
    const u64* list = list_array(P, 0u, row);
    if (j >= L.nb) {
        const TileCounts tiles{list_part<u32>(P, row, L.tile_off)};
        const u32 halves = (u32)((src_vectors<DT>(rs) + 2u * kLongBlock - 1u) / (2u * kLongBlock));
        auto ties = [&](u32 i) __attribute__((always_inline)) {
            if (L.half == 0) return tiles(i);
            return tiles(2u * i) + (2u * i + 1u < halves ? tiles(2u * i + 1u) : 0u);
        };
        if (mode == kListTied && done.total < rs.k &&
            !ties_of_row<DT, B, ListSource<DT, true>>(P, ties, row, rs, done.total, lr->T, j - L.nb, (u32)L.ties, sm.hist, sm.wsum) && j == L.nb && tid == 0)
            st->error |= 4u;  // never expected: there are enough of them
    } else if (bucket_range(P, L, row, rs, j, &at, &count) && count <= kBucketRoom) {
        const u64* src = list + at;
        order_in_lds<DT, B>(P, row, rs, sm, count, at, [&](u32 i) __attribute__((always_inline)) { return src[i]; });
    }
    if (done.big == 0u) return;
    // Every bucket that is too large is cut into parts of about half of what LDS holds, but into no more than there are workgroups, each part reading all of the bucket; all of the row's
    // parts are dealt to its workgroups.  (A row of 400000 fp32 keys, k = 9000, has 54 of them.  198013 of its entries in one bucket, in 97 parts, two to most workgroups, took 430 us; in 54, 267.)
    auto parts_of = [&](u32 count) __attribute__((always_inline)) {
        const u32 n = (count + 4u * B - 1u) / (4u * B);
        return n < per ? n : per;
    };
    if (j == 0u && tid == 0) st->redo |= kRedoBuckets;
    u32 base = 0;
    for (u32 j0 = 0; j0 < L.nb; j0 += B) {
        u32 n = 0;
        if (j0 + tid < L.nb && bucket_range(P, L, row, rs, j0 + tid, &at, &count) && count > kBucketRoom) n = parts_of(count);
        __syncthreads();
        const u32 incl = block_scan<B>(n, sm.wsum);
        before[tid] = incl - n;
        if (tid == B - 1) run = incl;
        __syncthreads();
        const u32 total = run;
        u32 W = per;
        asm volatile("" : "+s"(W));  // (its reciprocal is worked out here: kept from the kernel's beginning, every thread of every call wrote it to scratch memory, 262 KB of 2^28 keys' call)
        for (u32 s = (j + W - base % W) % W; s < total; s += W) {
            u32 a = 0, b = B;  // the bucket that part s belongs to: the last one that begins at or before it
            while (b - a > 1u) {
                const u32 m = (a + b) / 2u;
                if (before[m] <= s) a = m; else b = m;
            }
            bucket_range(P, L, row, rs, j0 + a, &at, &count);
            order_shared<DT, B>(P, row, rs, sm, shared, EntriesAt{list + at}, count, at, s - before[a], parts_of(count));
        }
        base += total;
    }
}

// ------------------------------------------------------------------------------------------------
// The kernels of a row that one workgroup takes alone, and those of rows that many share, are compiled apart (launch_list_rows_*, launch_list_*).
template <int DT, bool NT>
static void launch_row(const Params& P, const ListPlan& L, hipStream_t st) {
    const dim3 rows((unsigned)P.batch);
    if (L.row_block == 1024) hipLaunchKernelGGL((k_list_row<DT, 1024, 1, NT>), rows, dim3(1024), 0, st, P, L);
    else if (L.row_block == 512 && L.sample == 1) hipLaunchKernelGGL((k_list_row<DT, 512, 2, NT>), rows, dim3(512), 0, st, P, L);
    else if (L.row_block == 512) hipLaunchKernelGGL((k_list_row<DT, 512, 1, NT>), rows, dim3(512), 0, st, P, L);
    else if (L.sample == 1) hipLaunchKernelGGL((k_list_row<DT, 256, 4, NT>), rows, dim3(256), 0, st, P, L);
    else hipLaunchKernelGGL((k_list_row<DT, 256, 2, NT>), rows, dim3(256), 0, st, P, L);
}
template <int DT>
static void launch_rows(const Params& P, const ListPlan& L, hipStream_t st) {
    const dim3 rows((unsigned)P.batch);
    if (L.held == 0) {
        if (L.stream) launch_row<DT, true>(P, L, st);
        else launch_row<DT, false>(P, L, st);
    } else if (L.row_block == 128) hipLaunchKernelGGL((k_list_held<DT, 128, 4>), rows, dim3(128), 0, st, P, L);
    else if (L.row_block == 256 && L.held == 4) hipLaunchKernelGGL((k_list_held<DT, 256, 4>), rows, dim3(256), 0, st, P, L);
    else if (L.row_block == 256) hipLaunchKernelGGL((k_list_held<DT, 256, 8>), rows, dim3(256), 0, st, P, L);
    else if (L.row_block == 512 && L.held == 8) hipLaunchKernelGGL((k_list_held<DT, 512, 8>), rows, dim3(512), 0, st, P, L);
    else if (L.row_block == 512) hipLaunchKernelGGL((k_list_held<DT, 512, 16>), rows, dim3(512), 0, st, P, L);
    else hipLaunchKernelGGL((k_list_held<DT, 1024, 16>), rows, dim3(1024), 0, st, P, L);
}
template <int DT>
static rtopk_status launch_list_all(const Params& P, const ListPlan& L, hipStream_t st, void* const* events,
                                    void (*rows_alone)(const Params&, const ListPlan&, hipStream_t)) {
    mark(events, 0, st);
    mark(events, 1, st);
    const dim3 rows((unsigned)P.batch);
    if (L.row_block != 0) {
        mark(events, 2, st);
        mark(events, 3, st);
        rows_alone(P, L, st);
        mark(events, 4, st);
        return hipGetLastError() == hipSuccess ? RTOPK_OK : RTOPK_ERR_HIP;
    }
    if (L.seg_stride != 0) {
        hipLaunchKernelGGL((k_list_part<DT>), dim3((unsigned)P.batch * (unsigned)L.G), dim3(kPartBlock), 0, st, P, L);
        mark(events, 2, st);
        mark(events, 3, st);
        if (L.finish == 256) hipLaunchKernelGGL((k_part_finish<DT, 256>), rows, dim3(256), 0, st, P, L);
        else hipLaunchKernelGGL((k_part_finish<DT, 1024>), rows, dim3(1024), 0, st, P, L);
        mark(events, 4, st);
        return hipGetLastError() == hipSuccess ? RTOPK_OK : RTOPK_ERR_HIP;
    }
    const bool nt = L.stream != 0, is_long = L.nb != 0;
    const dim3 grid((unsigned)P.batch * (unsigned)L.G), block(L.stream_block != 0 ? L.stream_block : is_long ? kLongBlock : kGridBlock);
    if (L.stream_block != 0) {
        mark(events, 2, st);
        constexpr int kMost = DT == RTOPK_F32 ? 16 : 8;  // vectors per thread of the larger sample (16-bit keys: 16 do not fit the registers)
        auto sweep = [&](auto v, auto r) {
            if (nt) hipLaunchKernelGGL((k_list_stream<DT, decltype(v)::value, decltype(r)::value, true>), grid, block, 0, st, P, L);
            else hipLaunchKernelGGL((k_list_stream<DT, decltype(v)::value, decltype(r)::value, false>), grid, block, 0, st, P, L);
        };
        if (L.sample == 3) sweep(std::integral_constant<int, 8>{}, std::integral_constant<int, 8>{});
        else sweep(std::integral_constant<int, kMost>{}, std::integral_constant<int, 4>{});
    } else {
        if (L.sample == 2) hipLaunchKernelGGL((k_list_bound<DT, 512, 4>), rows, dim3(512), 0, st, P, L);
        else if (L.sample == 3) hipLaunchKernelGGL((k_list_bound<DT, 1024, 4>), rows, dim3(1024), 0, st, P, L);
        else if constexpr (DT == RTOPK_F32) {  // (16-bit keys: 16 vectors do not fit the registers)
            if (L.sample == 4) hipLaunchKernelGGL((k_list_bound<DT, 1024, 16>), rows, dim3(1024), 0, st, P, L);
            else hipLaunchKernelGGL((k_list_bound<DT, 1024, 8, 4>), rows, dim3(1024), 0, st, P, L);
        } else {
            hipLaunchKernelGGL((k_list_bound<DT, 1024, 8>), rows, dim3(1024), 0, st, P, L);
        }
        mark(events, 2, st);
        auto sweep = [&](auto nt_, auto long_) { hipLaunchKernelGGL((k_list_sweep<DT, decltype(nt_)::value, decltype(long_)::value>), grid, block, 0, st, P, L); };
        if (L.half != 0) hipLaunchKernelGGL((k_list_sweep<DT, false, true, 2>), grid, block, 0, st, P, L);
        else if (nt) is_long ? sweep(std::true_type{}, std::true_type{}) : sweep(std::true_type{}, std::false_type{});
        else is_long ? sweep(std::false_type{}, std::true_type{}) : sweep(std::false_type{}, std::false_type{});
    }
    mark(events, 3, st);
    if (is_long) {
        if (P.flags & RTOPK_FLAG_SORTED) hipLaunchKernelGGL((k_list_scatter<DT>), dim3(P.batch == 1 ? (unsigned)L.G + 1u : (unsigned)P.batch * (unsigned)L.G), block, 0, st, P, L);
        else hipLaunchKernelGGL((k_list_emit<DT>), grid, block, 0, st, P, L);
        hipLaunchKernelGGL((k_list_buckets<DT>), dim3((unsigned)P.batch * (L.nb + (unsigned)L.ties)), dim3(kListBucketBlock), 0, st, P, L);
    } else {
        const dim3 g((unsigned)P.batch * (1u + (unsigned)L.ties));
        if (L.stream_block != 0) hipLaunchKernelGGL((k_list_finish<DT, 1024, true>), g, dim3(1024), 0, st, P, L);
        else if (L.finish == 512) hipLaunchKernelGGL((k_list_finish<DT, 512, false>), g, dim3(512), 0, st, P, L);
        else hipLaunchKernelGGL((k_list_finish<DT, 1024, false>), g, dim3(1024), 0, st, P, L);
    }
    mark(events, 4, st);
    return hipGetLastError() == hipSuccess ? RTOPK_OK : RTOPK_ERR_HIP;
}

}  // namespace rtopk
