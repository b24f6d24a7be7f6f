// C-ABI entry points declared in include/rtopk.h: argument validation, the digit plan, workspace layout,
// and the hand-off to the per-type kernel launchers.  Host code, plus the one device object the library owns:
// the built-in scratch buffer of rtopk_select_static.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <atomic>
#include <mutex>

#include "rtopk.h"
#include "rtopk_device.h"
#include "rtopk_host.h"

namespace rtopk {

// ------------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------------
struct Layout {
    size_t state_off, dbg_off, ghist_off, seg_off, swg_off, sort_hist_off, sort_state_off, cand0_off, cand1_off, cand_stride, total;
};

static size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

static int elem_bytes(rtopk_dtype dt) { return dt == RTOPK_F32 ? 4 : 2; }

static rtopk_status make_config(int64_t batch, int64_t n, int64_t k, rtopk_dtype dt, int largest, uint32_t flags,
                                const rtopk_tuning* tn, Config* c) {
    if (batch < 1 || batch > 0x7fffffff || n < 1 || n > RTOPK_MAX_N || k < 1 || k > n) return RTOPK_ERR_INVALID_ARG;
    if (dt != RTOPK_F32 && dt != RTOPK_F16 && dt != RTOPK_BF16) return RTOPK_ERR_INVALID_ARG;
    if (flags & ~(uint32_t)(RTOPK_FLAG_SCALING | RTOPK_FLAG_DEBUG_COUNTERS | RTOPK_FLAG_SORTED)) return RTOPK_ERR_INVALID_ARG;
    int d = dt == RTOPK_F32 ? 12 : 11;
    int path = 0, G = 0;
    u32 small = 65536;
    if (tn) {
        if (tn->digit_bits) {
            if (tn->digit_bits < 8 || tn->digit_bits > 12) return RTOPK_ERR_INVALID_ARG;
            d = tn->digit_bits;
        }
        if (tn->path < 0 || tn->path > 3 || tn->wgs_per_row < 0 || tn->small_threshold < 0) return RTOPK_ERR_INVALID_ARG;
        path = tn->path;
        G = tn->wgs_per_row;
        if (tn->small_threshold) small = (u32)tn->small_threshold;
    }
    if (path == 0) {
        // short rows, or enough rows to occupy the compute units: one workgroup per row.  (fp32, k = 16 or 1024, row
        // kernel / grid kernels in us.  Uniform [0,1) keys, whose best bins are full: 1 x 2^15 32 / 36, 1 x 2^16
        // 45 / 36, 16 x 2^16 47 / 39, 64 x 2^16 46 / 45, 128 x 2^16 49 / 55, 1 x 2^18 86 / 50, 16 x 2^18 87 / 60,
        // 64 x 2^18 88 / 83, 128 x 2^18 90 / 107, 256 x 2^18 118 / 152.  Normal keys: 64 x 2^16 25 / 35,
        // 128 x 2^17 40 / 67, 256 x 2^18 100 / 130.)
        path = (n <= (1 << 16) || (batch >= 96 && n <= (1 << 18)) || (batch >= 256 && n <= (1 << 20))) ? 1 : 2;
        // ... unless a large part of every row is wanted: a workgroup that owns a row goes through its phases one
        // after the other (1024 rows of 2^17 bf16 keys, k = 8192: 51 + 36 us per row, 360 us in all), while the
        // grid kernels, one workgroup per row here, keep several rows per compute unit in flight (277 us; k = 2048:
        // 281 against 230, k = 1024: 217 against 224)
        if (path == 1 && batch >= 256 && batch <= 65535 && n >= 65536 && k * 128 >= n) path = 2;
        if (batch > 65535) path = 1;
    }
    // The one-sweep kernel sets aside a few hundred elements of a row (its bound comes from the row's first
    // eighth, more for larger k) and holds 2048.  Rows it cannot finish go to the two-sweep kernel, so the choice
    // never changes the result.  (A call without any knob takes lists for these shapes, see make_list_plan; the
    // automatic choice below is for calls that set another knob.)
    bool one_sweep = path == 3;
    if (path == 3) path = 1;
    // (k up to 512 on rows of 64K keys up: the bound then comes from a sample of the row and is checked afterwards --
    // 1024 rows of 2^17 bf16 keys, k = 1024: see the measurements beside the kernel)
    // (against the two-sweep row kernel, fp32, k = 16, in us: normal keys 128 x 2^17 32 / 40, 256 x 2^17 41 / 57,
    // 256 x 2^18 60 / 100, 512 x 2^17 63 / 102; uniform [0,1) keys, where the first part shows a full bin at the top and
    // most rows are handed over: 256 x 2^16 61 / 55, 256 x 2^18 123 / 118.  With fewer rows than a quarter of the
    // compute units there is nothing to overlap: 16 x 2^16 uniform keys 47 / 41, 64 x 2^16 normal keys 24 / 25.)
    else if (path == 1 && (!tn || tn->path == 0) && (k <= 256 || (k <= 512 && n >= 65536)) && n >= 16384 && batch >= 64)
        one_sweep = true;
    if (path == 2 && batch > 65535) return RTOPK_ERR_INVALID_ARG;  // rows are the grid's y dimension
    // 16-bit keys on long rows: a 12-bit first digit (4 bits left for the second) instead of 11 + 5 -- the first
    // sweep then keeps a bin of half the width (bf16 logits, 64 x 2^22, k = 50: 200 -> 167 us; 2^29 uniform bf16
    // keys: 1052 -> 788 us); the one-workgroup-per-row kernels stay at 11, where twice the histogram copies fit
    // (not where one workgroup has a whole row of such a batch and k is small: 1024 rows of 2^17 bf16 keys, 11 against
    // 12 bits: k = 1024 203 against 222 us, k = 2048 222 against 230, k = 4096 290 both, k = 8192 283 against 276)
    if (path == 2 && dt != RTOPK_F32 && !(tn && tn->digit_bits) && !(batch >= 256 && k * 32 <= n)) d = 12;
    const int eb = elem_bytes(dt);
    const int64_t tile_elems = (int64_t)kHostGridBlock * kHostElemsPerLane;  // 16 elements per lane for every type
    const int64_t ntiles = (n + 16 / eb - 1 + tile_elems) / tile_elems;  // one spare for the lead-in
    // Prefilter (many workgroups per row, unscaled): count a sample of the row (every 31st tile: a prime stride,
    // so that no power-of-two period in the data lines up with the sample), take from it a bin that very
    // probably lies at or below the k-th key's, and sweep X ONCE, counting every element's digit and keeping the
    // elements from that bin upwards; pass 0 then runs on what was kept.  If the full counts show the bin was
    // too high, pass 0 is the ordinary second sweep over X instead.
    // It pays while k is well below n (what is kept is written out and read again): 2^28 uniform fp32 keys,
    // k = 2^24 (a sixteenth: 9 % of the row kept) 395 us against 526 with two sweeps; from k = 2^25 on the sample
    // shows more than an eighth of the row in the bins to keep and the sweep would decline anyway.
    c->prefilter = false;
    c->pre_stride = 0;
    if (tn && (tn->prefilter < -1 || tn->prefilter > 1)) return RTOPK_ERR_INVALID_ARG;
    const int pre_knob = tn ? tn->prefilter : 0;
    const bool scaling_on = (flags & RTOPK_FLAG_SCALING) && dt == RTOPK_F32;
    // (inputs of 64 to 256 MB: two sweeps from the caches cost little more than one, and the call is bound by its
    // launches; for fp32 keys the prefilter still wins where pass 0 would otherwise write many candidates -- 2^24
    // normal keys, k = 2^16: 62 against 82 us, k = 2^12: 61 against 65, k = 16: 61 against 56 -- and for batches,
    // whatever k: 16 rows of 2^20, k = 16: 79 against 106; 64 rows of 2^20: 132 against 189; 2^26 fp16 keys that
    // all fall into one bin lost 100 us to the counting sweep that then stands before the two others)
    const int64_t in_bytes = batch * n * eb;
    // (up to a sixteenth of the row for fp32 inputs of 256 MB up; a 32nd otherwise: 2^24 fp32 keys, k = 2^20: 93 against
    // 83 us; 1024 rows of 2^17 bf16 keys, k = 2^13: the sample declines, 298 against 273 us)
    const bool big_f32 = dt == RTOPK_F32 && in_bytes >= ((int64_t)256 << 20);
    if (path == 2 && !scaling_on &&
        (pre_knob == 1 || (pre_knob == 0 && k <= n / (big_f32 ? 16 : 32) &&
                           (in_bytes >= ((int64_t)256 << 20) ||
                            (dt == RTOPK_F32 && in_bytes >= ((int64_t)64 << 20) && (batch > 1 || k * 4096 >= n)))))) {
        c->prefilter = true;
        c->pre_stride = 31;
    }
    if (path == 2) {
        if (G == 0) {
            // about two workgroups per compute unit in total; one for the fp32 sweep that counts and keeps, which
            // then stages three times as much per wave (measured on n = 2^28: k = 2^20 239 us with 256 workgroups,
            // 280 with 512, 298 with 384; k = 2^22 321 against 332; k = 2^24 389 against 395; two sweeps with
            // k = 2^24: 603 against 526)
            // (16-bit keys: whole bins of an 11-bit digit are kept, more of the row; 2^29 fp16 keys, k = 2^20:
            // 260 us with 512, 346 with 256; bf16 with k = 50 or 2^10: no difference)
            // (and one for inputs that the caches hold: 2^24 fp32 keys, two sweeps: 53-61 us against 58-65; not
            // 128 MB: 2^26 fp16 keys of few distinct values, 355-385 us against 270-303)
            const bool cached = in_bytes <= ((int64_t)64 << 20);
            int64_t want = ((c->prefilter && dt == RTOPK_F32) || cached ? 256 : 512) / batch;
            if (want < 1) want = 1;
            G = (int)want;
        }
        if (G > ntiles) G = (int)ntiles;
        if (G > 4096) G = 4096;
        if (G < 1) G = 1;
    } else {
        G = 1;
    }
    // sorted output of rows too long for one workgroup's LDS: a radix sort on the grid, chunks of at least 8192 keys
    c->Gs = 0;
    if ((flags & RTOPK_FLAG_SORTED) && k > kHostSortSmall) {
        int64_t want = 512 / batch, by_k = (k + 8191) / 8192;
        if (want < 1) want = 1;
        if (want > by_k) want = by_k;
        c->Gs = (int)want;
        if (batch > 65535) return RTOPK_ERR_INVALID_ARG;  // rows are the grid's y dimension there
    }
    c->d = d;
    c->path = path;
    c->one_sweep = one_sweep;
    c->G = G;
    c->small = small;
    c->dirmask = largest ? 0u : (dt == RTOPK_F32 ? 0xffffffffu : 0xffff0000u);

    int np = 0;
    const int kw = dt == RTOPK_F32 ? 32 : 16;
    if ((flags & RTOPK_FLAG_SCALING) && dt == RTOPK_F32) {
        for (int hi = 32; hi > 0;) {
            int bits = d < hi ? d : hi;
            c->pass[np++] = PassInfo{SRC_SCALED, (u32)(hi - bits), (u32)bits};
            hi -= bits;
        }
    }
    for (int hi = 32; hi > 32 - kw;) {
        int bits = d < hi - (32 - kw) ? d : hi - (32 - kw);
        c->pass[np++] = PassInfo{SRC_KEY, (u32)(hi - bits), (u32)bits};
        hi -= bits;
    }
    int ib = 0;
    while (((int64_t)1 << ib) < n) ++ib;
    c->idx_max = ib == 0 ? 0u : (u32)(((u64)1 << ib) - 1);
    for (int hi = ib; hi > 0;) {
        int bits = d < hi ? d : hi;
        c->pass[np++] = PassInfo{SRC_IDX, (u32)(hi - bits), (u32)bits};
        hi -= bits;
    }
    if (np > kMaxPasses) return RTOPK_ERR_INVALID_ARG;
    c->npass = np;
    // How far can a row keep more than `small` candidates?  Key digits may keep all n (equal keys); after an
    // index digit at most 2^shift candidates share the bin, the indices being distinct.  Later passes are
    // certain to fit the single-workgroup finish and get no grid launch.
    c->multi_last = np - 1;
    for (int p = 0; p < np; ++p) {
        const bool idx = c->pass[p].src == SRC_IDX;
        const uint64_t bound = idx && c->pass[p].shift < 63 && ((uint64_t)1 << c->pass[p].shift) < (uint64_t)n
                                   ? (uint64_t)1 << c->pass[p].shift : (uint64_t)n;
        if (bound <= small) {
            c->multi_last = p;
            break;
        }
    }
    return RTOPK_OK;
}

static Layout make_layout(int64_t batch, int64_t n, const Config& c) {
    Layout L;
    size_t off = 0;
    L.state_off = off;
    off = align_up(off + (size_t)batch * RTOPK_TRACE_STRIDE, 256);
    L.dbg_off = off;
    off = align_up(off + (size_t)batch * c.G * 128, 256);
    // global histograms, per-workgroup records and segments exist only when several workgroups share a row
    const size_t shared_rows = c.path == 2 ? (size_t)batch : 0;
    L.ghist_off = off;
    off = align_up(off + (size_t)kHostHistBuffers * shared_rows * kMaxBins * 4, 256);
    L.seg_off = off;
    off = align_up(off + (size_t)2 * shared_rows * c.G * 2 * 4, 256);
    L.swg_off = off;
    off = align_up(off + (size_t)kHostSwgBuffers * shared_rows * c.G * kSwgStride * 4, 256);
    L.sort_hist_off = off;
    off = align_up(off + (size_t)batch * 256 * c.Gs * 4, 256);
    L.sort_state_off = off;
    off = align_up(off + (c.Gs ? (size_t)batch * 128 : 0), 256);
    // (the prefilter's per-workgroup segments are laid out by whole tiles: up to two tiles beyond n)
    L.cand_stride = (size_t)n + (c.prefilter ? (size_t)2 * kHostGridBlock * kHostElemsPerLane : 0);
    L.cand0_off = off;
    off = align_up(off + (size_t)batch * L.cand_stride * 8, 256);
    L.cand1_off = off;
    off = align_up(off + (size_t)batch * L.cand_stride * 8, 256);
    L.total = off + 256;  // the last 16-byte load of an odd-length candidate array may touch 8 bytes past it
    return L;
}

// Does the call go through lists (rtopk_list.inl), and how?  The automatic choice only: a call with tuning knobs gets the
// kernels it names.
static bool make_list_plan(int64_t batch, int64_t n, int64_t k, rtopk_dtype dt, const rtopk_tuning* tn, bool ragged, bool sorted,
                           ListPlan* L) {
    memset(L, 0, sizeof(*L));
    if (tn && (tn->digit_bits || tn->path || tn->wgs_per_row || tn->small_threshold || tn->prefilter)) return false;
    const int eb = elem_bytes(dt), E = 16 / eb;
    // Few rows above 128 KB, k of at most 64: stretches of 32 KB, each listing its best k.  us, rows held whole / in stretches:
    // 16 rows of 2^17 bf16 keys, k = 50, 23.8 / 15.2, 96 rows 27.3 / 21.1, one fp32 row of 2^16, k = 10, 14.0 / 11.9.  With a
    // large k the stretches' lists are most of the work (16 rows of 2^16 fp32 keys, k = 300, 16.7 / 20.2; 96 rows of 2^17
    // bf16 keys 28.7 / 30.6), and a short row is held by 256 or 512 threads, in one launch (16 fp32 rows of 20000, k = 10, 11.5 / 12.5;
    // 48 bf16 rows of 50257, k = 50, 18.9 / 21.2).  Rows off the 16-byte grid have stretches with lanes that are partly empty and
    // bound less: 16 fp32 rows of 50000, k = 32, 15.0 / 12.8, but of 50257 16.1 / 18.6; 16-bit keys have more to a lane and win
    // up to k = 50 (48 bf16 rows of 100003 27.2 / 23.3; a single one, k = 64, 22.2 / 23.4).
    {
        const int64_t part = (int64_t)kListPartBlock * kListPartVecs * 16, G = (n * eb + 16 + part - 1) / part;
        const int64_t stride = k * 2 + 64;
        const bool whole = !ragged && n % E == 0;
        if (k <= (whole ? 64 : eb == 2 ? 48 : 0) && n * eb > (128 << 10) && batch * G <= 1024 && G * stride <= 8192) {
            L->G = (int)G;
            L->seg_stride = (u32)stride;
            L->finish = G * stride <= 2048 ? 256 : 1024;
            L->seg_off = kListMetaBytes;
            return true;
        }
    }
    // rows that one workgroup can hold in registers
    if (batch <= ((int64_t)1 << 22)) {
        static const struct { int block, vecs; int64_t rows; } held[] = {
            {128, 4, 1 << 22}, {256, 4, 1 << 22}, {256, 8, 1 << 22}, {512, 8, 1 << 22}, {512, 16, 512}, {1024, 16, 256}};
        for (const auto& h : held) {
            if (n * eb > (int64_t)h.block * h.vecs * 16) continue;
            if (n > 8 * h.block && k + k / 16 + 2 > 8 * h.block) continue;  // the list's room
            if (n > 8 * h.block && h.vecs == 16 && k > h.block / 2) continue;  // (bounded by the lanes' best elements only)
            if (batch > h.rows) break;
            // Unsorted output of a larger part of a row: the list is ranked for nothing, the digit passes write their winners as they
            // find them (in one launch as well).  us, digit passes / list, normal keys: one fp32 row of 4096, k = 100 12 / 9, k = 409 13 / 12,
            // k = 1000 13 / 17, of 16384, k = 1000 17 / 15, k = 4915 20 / 20; keys of 100 values, k = 1228 of 4096, 13 / 47.  16-bit keys, whose
            // vectors' maxima bound less: 4096, k = 40 11 / 9, k = 100 11 / 13, k = 409 11 / 23; 16384, k = 100 12 / 11, k = 1638 15 / 31.  Many
            // rows: a smaller workgroup per row wins by far up to a quarter of the row (1024 fp32 rows of 4096, k = 1228, 58 / 26; 1024 fp16
            // rows of 16384, k = 1638, 69 / 54, k = 4915 61 / 88).
            if (!sorted && (batch <= 512 ? k * (eb == 4 ? 16 : 64) > n : n > 8192 && k * 4 > n)) return false;
            L->row_block = h.block;
            L->held = h.vecs;
            return true;
        }
    }
    // The same for rows that one workgroup sweeps: one fp32 row of 16384, k = 4915, 20 / 23, of 30000, k = 3000, 26 / 24; fp16 rows of 30000,
    // k = 3000, 23 / 31, of 50257, k = 5025, 38 / 33.
    if (!sorted && batch <= 512 && n <= 40000 && k * (eb == 4 ? 4 : 16) > n) return false;
    // the smallest sample is 8 KB of a row, a quarter of 32 KB
    if (n * eb < 32768) return false;
    // the list is to stay below half the row (in a ragged batch: half the longest row, for every row)
    if (k * 5 > (ragged ? n : n * 2)) return false;
    // A list's 4096 bins hold more than a workgroup puts in order once k is in the millions.  Digit passes / list, us, 2^28 fp32
    // keys: sorted, k = 2^22, 1120 / 317, 2^23 1479 / 1370, 2^24 2460 / 2362; unsorted, k = 2^21, 456 / 356, 2^22 442 / 487,
    // 2^24 586 / 2694.
    if (k > ((int64_t)1 << (sorted ? 22 : 21))) return false;
    const int64_t vecs = n * eb / 16;
    L->sample = vecs >= (1 << 20) ? 4 : vecs >= (1 << 16) ? 3 : vecs >= (1 << 14) ? 2 : vecs >= (1 << 12) || batch <= 256 ? 1 : 0;
    // one workgroup per row: rows of up to 256 KB, in large batches up to 1 MB
    const bool by_row = n * eb <= (256 << 10) || (batch >= 256 && n * eb <= (1 << 20));
    if (by_row && L->sample > 1) L->sample = 1;
    double listed = 0.0, room = 0.0;  // expected length of the list, and with a margin
    auto expect = [&](int64_t sampled) {
        const double elems = (double)(sampled * E);
        const double ks = (double)k * elems / (double)n;
        listed = (ks + 6.0 * __builtin_sqrt(ks) + 7.0) * 1.08 * (double)n / elems;
        room = listed * 1.08 + 64.0;
    };
    auto sample_vecs = [&]() { return L->sample == 4 ? (eb == 4 ? 16384 : 8192) : L->sample == 3 ? 4096 : 512 << L->sample; };
    expect(sample_vecs());
    if (by_row) {
        // (a list that does not fit is put in order part by part: better a little too much room)
        L->row_block = batch > 256 && room * 1.2 <= 2048.0 ? 256 : batch > 256 && room * 1.2 <= 4096.0 ? 512 : room <= 8192.0 ? 1024 : 0;
        if (L->row_block == 1024 && L->sample == 0) L->sample = 1;
    }
    if (L->row_block == 0 && L->sample < 2) {  // (the kernels for many workgroups per row take larger samples)
        if (vecs < 4096) return false;
        L->sample = 2;
    }
    // Short lists of few rows: sample and sweep in one launch (k_list_stream), with half the sample, while one workgroup puts in order what that lists
    // (up to twice as much as it should be, 16384 entries at most).  us, two launches / one, normal keys: one fp32 row of 1.5 million, k = 16, 300 and 3000,
    // 22.2 / 20.0, 25.1 / 21.5, 30.9 / 27.4; of 2^23 keys, k = 16, 100 and 256, 34.7 / 26.6, 36.3 / 28.0, 33.6 / 29.3; of 24 million 42.3 / 37.0,
    // 44.4 / 38.9, 44.2 / 42.6.  fp16 rows of 2 million 22.4 / 21.0, 26.5 / 21.8, 33.3 / 28.6.
    // Rows below 1 MB have a sample of 2048 vectors in a launch of its own, half of the one that is taken here, which every workgroup has to rank: fp32 rows of 2^17, k = 300,
    // one 21.1 / 21.0, 8 20.3 / 23.4, 24 23.4 / 30.1; of 200000, k = 300 and 1500, one 21.5 / 21.8, 24.8 / 28.1, 8 22.9 / 23.6, 25.8 / 34.4; of 2^18 one 22.5 / 20.5, 25.5 /
    // 23.3, 8 23.2 / 21.1, 26.8 / 24.7; eleven of 135112, k = 615, 22.5 / 30.2.  16-bit rows of 1 MB gain as much with normal keys (one of 2^19 22.5 / 19.9), but not
    // a ramp with infinities (42 / 56); from 3 MB on that is gone (1.6 million 52.9 / 52.2).
    // 16-bit keys have twice the arithmetic per byte, and the two launches twice the waves to hide it behind, where ties are counted above all: one bf16 row of 16 million, nine
    // in ten equal, 30.7 / 32.8; 32 rows of 1.7 million fp16 keys, k = 16, normal 38.4 / 38.9, nine in ten equal 45.5 / 51.0, uniform, k = 300, 56.9 / 43.4; 30 of 2^21
    // 41.2 / 44.2, 40.9 / 44.4, 57.0 / 46.1; 32 of 2^21 43.2 / 47.8, 50.7 / 60.9, 58.1 / 51.3.
    // More than 32 rows have so few workgroups each that they take the sample for little: 24 fp32 rows of 2^18, k = 300, 27.5 / 24.6, 32 27.6 / 26.8, 40 29.6 / 27.5, 64
    // 31.2 / 32.2; of 2^19 32 33.5 / 31.9, 64 43.9 / 50.6.  (32 fp32 rows of 2^20, 4 MB apart, eight workgroups each: k = 16 44.1 / 46.0, k = 300 54.0 / 48.4; 28 rows 39.5 / 36.4,
    // 48.4 / 38.7, 32 of 10^6 38.9 / 38.7, 47.4 / 41.4.)
    bool stream = false;
    if (L->row_block == 0 && batch <= 32 && n * eb >= ((int64_t)(eb == 4 ? 1 : 3) << 20) &&
        (eb == 4 || (n * eb <= ((int64_t)24 << 20) && batch * n * eb <= ((int64_t)112 << 20)))) {
        expect(L->sample == 4 && eb == 4 ? 8192 : 4096);
        stream = room <= 8192.0 && listed * 1.1 <= 0.5 * (double)n;
    }
    if (!stream) expect(sample_vecs());
    if (listed * 1.1 > 0.5 * (double)n) return false;
    const bool is_long = L->row_block == 0 && !stream && room > 8192.0;
    // A long list's bound comes from half the largest sample: the one workgroup that takes it needs 6 to 7 us to fetch all of it and as long to rank and gather it, and the row's list
    // is only a tenth longer where k is large.  It has as many runs as all of it, half as long: with half as many, trends' lists and bins come out up to twice as long.  240 rows of 2^22 to
    // 2^27 keys, k from 1000 up, half the runs / this, each against all of the sample's time (geometric mean): normal keys 0.92 / 0.93; nine in ten equal 0.90 / 0.91; a thousand values
    // 0.95 / 0.97; ramps 1.09 / 0.99; with infinities 0.99 / 0.95; blocks of 64 equal neighbours 1.08 / 0.94; single calls, whose T falls a run lower or higher, up to 1.8 and down to 0.6.  (A quarter
    // gains 1 to 3 us more on normal keys, but 2^28 uniform ones, k = 2^20, 229.5 / 243.4.)
    if (is_long && L->sample == 4 && eb == 4) {
        expect(8192);
        if (listed * 1.1 > 0.5 * (double)n) expect(sample_vecs());
        else L->sample = 5;
    }
    // Unsorted long lists: what lies above rank k's bin is output as it comes, and that bin alone is ordered.  fp32 rows of 2^25 keys and more go that way; the rest is left to the digit passes, a line that was drawn
    // when all of the list was put in order.  As it is now the list gains wherever keys are in no order, and loses where they lie in order along the row and crowd a few tiles.  One row, us, digit passes / list, k = n /
    // 1000, n / 100 and n / 16: 2^22 fp32 keys, normal, 42 / 34, 53 / 35, 69 / 41, nine in ten equal 88 / 40, 88 / 52, 88 / 84, ramps with infinities 53 / 70, 56 / 78, 57 / 83; 2^26 fp16 keys, k = n / 1000 and n / 100, 91 /
    // 57, 119 / 59, equal 249 / 82, 249 / 87, ramps 134 / 170, 127 / 192; 2^24 bf16 keys 62 / 43, 68 / 44, 79 / 59, equal 122 / 53, 123 / 64, 123 / 117, ramps 84 / 168, 85 / 156, 87 / 179.
    if (is_long && !sorted && (eb != 4 || n < ((int64_t)1 << 25))) return false;
    // k_list_stream: a workgroup of 512 threads per compute unit; k_list_sweep: one of 1024 where the list's histogram is counted, else four
    // of 512 (three for 16-bit keys), but no more than 256 to a row, 512 for 16-bit keys up to 128 MB.  The more there are, the more segments have to be put together, and the
    // fewer, the less is there to hide the arithmetic of counting ties behind, of which 16-bit keys have twice as much.
    // us, 1024 (16-bit keys: 768) / 512 / 256 to a row: one fp32 row of 2^25, k = 16 and 300, 51.5 / 50.1 / 49.5 and 50.9 / 50.7 / 50.6, of 3 * 2^24, k = 16, 59.1 / 58.0 /
    // 56.4; one of 2^25 fp16 keys, k = 100, 41.1 / 38.5 / 37.9, nine in ten equal 42.5 / 43.6 / 48.1; of 14 million, nine in ten equal, 34.6 / 34.9 / 38.4;
    // of 2^24 bf16 keys, a ramp, k = 100, 55.4 / 56.7 / 58.4; of 2^26, k = 300, nine in ten equal, 62.7 / 64.7 / 64.2.
    // A single row of up to 8.5 MB has no more than 136 tiles of 64 KB for 256 compute units: a long list's sweep takes half as large ones there, and the histograms of then up to 256 workgroups,
    // which all end together, are added up in four copies (an add to a line of counters takes 11 ns).  us, tiles of 64 KB / of 32, one histogram / so: 2^22 + 3 fp16 keys, k = 2^20,
    // 58.3 / 55.9 / 54.1; 2^21 fp32 keys, k = 20000 31.9 / 34.1 / 32.2, k = n / 5 41.2 / 42.3 / 40.2; 2^18 fp32 keys, k = n / 5 36.1 / 33.5 / 34.0; ramps, whose list lies in a few tiles, 2^21, k =
    // 20000, 110 / 80, 2^20 fp16 keys 117 / 94.  Nine in ten equal 2^20 fp32 keys, k = 10000 and n / 4, 34.0 / 35.8 and 57.6 / 59.5.  At 8 MB each compute unit has one tile of 32 KB, and the line lies half a megabyte
    // above that for rows of a power of two and a few more; it is not a sharp one: from 8.1 to 12 MB some workgroups have two tiles and others one, normal keys take the same time either way (2^21 + 2^15 fp32 keys, k =
    // 20000, 32 / 32, 9 MB of fp16 keys, k = n / 4, 62 / 62), equal ones 2 to 3 us more (40 / 43, 47 / 50) and ramps a quarter less (110 / 82, 158 / 118).
    L->half = is_long && batch == 1 && n * eb <= ((int64_t)17 << 19) ? 1 : 0;
    const int64_t tile_elems = (int64_t)(is_long && L->half == 0 ? 1024 : kHostGridBlock) * 64 / eb;
    const int64_t ntiles = (n + E - 1 + tile_elems - 1) / tile_elems;
    const int64_t wave_tiles = (n + E - 1 + 256 * E - 1) / (256 * E);  // (k_list_stream's)
    int64_t G = (stream || is_long ? 256 : eb == 4 ? 1024 : 768) / batch;
    if (G < 1) G = 1;
    if (G > (stream ? wave_tiles : ntiles)) G = stream ? wave_tiles : ntiles;
    const int64_t most_wgs = eb == 2 && batch * n * eb < ((int64_t)128 << 20) ? 512 : 256;
    if (!is_long && G > most_wgs) G = most_wgs;
    L->G = (int)G;
    L->stream_block = stream ? 512 : 0;
    // (one sweep: nothing is read twice.  2^26 fp32 keys, k = n / 100 as a mask, 133 us with ordinary loads, 121 past the
    // caches; 1024 rows of 2^17 bf16 keys, k = 50, 64 against 57.5; 2^24 fp32 keys, which the last-level cache holds, 36.7
    // against 37.8)
    L->stream = batch * n * eb > ((int64_t)128 << 20);
    // (256 segments to read keep 1024 threads busy: one fp16 row of 6 million, k = 16, 256 threads 25.9, k = 100, 1024 threads 23.3.  512 threads take no longer than 256 for a list as
    // long as expected, 64 rows of 2^18 fp16 keys, k = 300, 21.6 / 21.5, and longer ones in half the time (see k_list_finish).  One of more than 2048 entries is cut down first, so a little
    // too much room here as well: 32 rows of 2^21 fp16 keys, k = 300, room for 1907 entries, 54.7 / 50.1)
    L->finish = room * 1.2 > 2048.0 || stream || G > 256 ? 1024 : 512;  // (and a thread per segment)
    L->room = L->finish == 512 ? 2048u : 8192u;
    const double twice = 2.0 * room < 2.0 * L->room ? 2.0 * room : 2.0 * L->room;
    L->most = twice > L->room ? (u32)twice : L->room;
    // (Twice the average segment's entries; less where they are a hundred and more, whose number varies less: places that stay empty are read for
    // nothing.  One row of 131072 fp32 keys, nine in ten equal, k = 1000, 21.1 us with twice as many, 20.4 so; but one of 14 million fp16 keys, k = 16, in 256 short segments,
    // 31.9 / 34.4.  No more than 16 places per thread, and not most of the row's working memory.)
    const double places = room >= 64.0 * (double)G ? 1.4 * room : 2.0 * room;
    L->slots = 8;
    while ((double)L->slots * (double)G < places && (int64_t)L->slots * 2 * G <= (int64_t)L->finish * 16 && (int64_t)L->slots * 16 * G <= n * 2) L->slots *= 2;
    if (is_long || L->row_block != 0) L->slots = 0;
    L->bucket_shift = 11;
    while ((k >> L->bucket_shift) + 1 > (int64_t)kListMaxBuckets) ++L->bucket_shift;
    L->nb = !is_long ? 0u : sorted ? (u32)((k >> L->bucket_shift) + 1) : 1u;  // (unsorted: one, for the bin that rank k lies in)
    int64_t ties = 128 / batch;
    if (ties < 1) ties = 1;
    if (ties > ntiles) ties = ntiles;
    L->ties = (int)ties;
    if (batch * ((int64_t)L->nb + 1 + ties) >= ((int64_t)1 << 22) || batch * G >= ((int64_t)1 << 22)) return false;  // grid sizes
    u64 off = kListMetaBytes;
    // (whole cache lines: a wave's adds to 64 neighbouring counters fall on two of them, not three -- 4 million fp16 keys, k = 2^20, 64.8 / 62.3 us)
    auto take = [&](u64 bytes) { const u64 at = off; off = align_up(off + bytes, 128); return (u32)at; };
    L->front_off = take((u64)G * L->slots * 8);
    L->seg_off = take((u64)G * 8);
    L->hists = L->half != 0 && G > 64 ? 4u : 1u;
    L->hist_off = take(is_long ? (u64)L->hists * kMaxBins * 4 : 0);
    L->cursor_off = take(is_long ? (u64)list_cursors(L->nb) * 8 : 4);
    L->first_off = take((u64)L->nb * 8);
    L->split_off = take(is_long ? (kListSplits + 1) * 8 : 0);
    L->tile_off = take((u64)(stream ? wave_tiles + 2 : (n + E - 1) / (kHostGridBlock * 64 / eb) + 2) * 4);  // (the smallest tiles' number)
    L->stack_off = take(((u64)n / 256 + 64 + 16 * (u64)L->nb) * 16);
    return off + 256 + 8 <= (u64)n * 4;  // (the upper half of a candidate array)
}

}  // namespace rtopk

using namespace rtopk;

// The scratch memory of rtopk_select_static: part of the device code, one copy per GPU.  In host code this
// name is only a handle for hipGetSymbolAddress; kernels and copies get the address looked up below.
static __device__ __align__(256) unsigned char scratch[RTOPK_STATIC_SCRATCH_BYTES];

// Address of `scratch` on the current device, looked up once per device (each GPU has its own copy at its own
// address).  Returns nullptr if the runtime cannot tell.
static void* static_scratch_of_current_device() {
    constexpr int kMaxDevices = 64;
    static std::atomic<void*> known[kMaxDevices];
    static std::mutex lookup;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    void* p = known[dev].load(std::memory_order_acquire);
    if (p) return p;
    std::lock_guard<std::mutex> hold(lookup);
    p = known[dev].load(std::memory_order_relaxed);
    if (!p) {
        void* found = nullptr;
        if (hipGetSymbolAddress(&found, HIP_SYMBOL(scratch)) != hipSuccess || !found) return nullptr;
        p = found;
        known[dev].store(p, std::memory_order_release);
    }
    return p;
}

// How much of a streamed row (its tail) the first sweep reads with cache-allocating loads, for the second sweep
// to find in the caches (MI355X: 256 MB last-level cache + 32 MB of L2).  Measured on n = 2^28 fp32: the whole call takes
// 462 us with nothing kept, 449 with 256 MB, 444-445 with 288-320 MB, 451 with 352 MB and more (the first sweep
// slows down by more than the second gains).
static const size_t kKeepBytes = (size_t)288 << 20;

extern "C" {

const char* rtopk_status_string(rtopk_status s) {
    switch (s) {
        case RTOPK_OK: return "ok";
        case RTOPK_ERR_INVALID_ARG: return "invalid argument";
        case RTOPK_ERR_WORKSPACE_TOO_SMALL:
            return "workspace too small for these arguments and tuning (size it with rtopk_workspace_bytes_ex and the same tuning)";
        case RTOPK_ERR_UNSUPPORTED: return "unsupported (misaligned buffer)";
        case RTOPK_ERR_HIP: return "HIP runtime rejected a launch";
        case RTOPK_ERR_STATIC_SCRATCH:
            return "these arguments need more scratch memory than the built-in buffer of rtopk_select_static holds "
                   "(RTOPK_STATIC_SCRATCH_BYTES); use rtopk_select with a caller-owned workspace";
    }
    return "unknown status";
}

const char* rtopk_version(void) { return "0.1"; }

rtopk_status rtopk_workspace_bytes_ex(int64_t batch, int64_t n, int64_t k, rtopk_dtype dt, uint32_t flags,
                                      const rtopk_tuning* tuning, size_t* bytes_out) {
    if (!bytes_out) return RTOPK_ERR_INVALID_ARG;
    Config c;
    rtopk_status s = make_config(batch, n, k, dt, 1, flags, tuning, &c);
    if (s != RTOPK_OK) return s;
    *bytes_out = make_layout(batch, n, c).total;
    return RTOPK_OK;
}

rtopk_status rtopk_workspace_bytes(int64_t batch, int64_t n, int64_t k, rtopk_dtype dt, uint32_t flags,
                                   size_t* bytes_out) {
    return rtopk_workspace_bytes_ex(batch, n, k, dt, flags, nullptr, bytes_out);
}

// Every entry point ends here.  row_offsets / row_k: null, or the ragged batch's device arrays (n and k are then the
// largest row length and the largest k).
static rtopk_status select_impl(const void* keys, const int64_t* row_offsets, const int64_t* row_k, int64_t batch, int64_t n,
                                int64_t k, rtopk_dtype dt, int largest, uint32_t flags, uint64_t seed, void* out_values,
                                int64_t* out_indices, void* workspace, size_t workspace_bytes, void* hip_stream,
                                const rtopk_tuning* tuning, void* const* events) {
    if (!keys || !out_values || !out_indices || !workspace) return RTOPK_ERR_INVALID_ARG;
    if ((row_offsets == nullptr) != (row_k == nullptr)) return RTOPK_ERR_INVALID_ARG;
    Config c;
    rtopk_status s = make_config(batch, n, k, dt, largest, flags, tuning, &c);
    if (s != RTOPK_OK) return s;
    const int eb = elem_bytes(dt);
    if (((uintptr_t)keys % eb) || ((uintptr_t)out_values % eb) || ((uintptr_t)out_indices % 8) ||
        ((uintptr_t)workspace % 256))
        return RTOPK_ERR_UNSUPPORTED;
    const Layout L = make_layout(batch, n, c);
    if (workspace_bytes < L.total) return RTOPK_ERR_WORKSPACE_TOO_SMALL;

    Params P;
    memset(&P, 0, sizeof(P));
    char* ws = (char*)workspace;
    P.keys = keys;
    P.row_offsets = (const long long*)row_offsets;
    P.row_k = (const long long*)row_k;
    P.out_values = out_values;
    P.out_indices = (long long*)out_indices;
    P.state = (rtopk_row_trace*)(ws + L.state_off);
    P.ghist = (u32*)(ws + L.ghist_off);
    P.seg = (u32*)(ws + L.seg_off);
    P.dbg = (unsigned long long*)(ws + L.dbg_off);
    P.swg = (u32*)(ws + L.swg_off);
    P.sort_hist = (u32*)(ws + L.sort_hist_off);
    P.sort_state = (void*)(ws + L.sort_state_off);
    P.Gs = c.Gs;
    P.cand[0] = (uint2*)(ws + L.cand0_off);
    P.cand[1] = (uint2*)(ws + L.cand1_off);
    P.cand_stride = L.cand_stride;
    P.pre_stride = c.prefilter ? c.pre_stride : 0u;
    P.n = n;
    P.k = k;
    P.batch = (int)batch;
    P.G = c.G;
    P.dirmask = c.dirmask;
    P.idx_max = c.idx_max;
    P.small = c.small;
    P.npass = c.npass;
    P.flags = flags;
    // two sweeps over more data than the 256 MB last-level cache holds: stream it past the caches
    P.keep_from_tile = 0xffffffffu;
    if ((size_t)batch * (size_t)n * (size_t)eb > ((size_t)384 << 20)) {
        P.flags |= kInternalStream;
        // a single long row: leave its last kKeepBytes in the last-level cache for the second sweep
        const size_t tile_bytes = (size_t)kHostGridBlock * kHostElemsPerLane * eb;
        const size_t row_tiles = ((size_t)n * eb + tile_bytes - 1) / tile_bytes;
        const size_t keep_tiles = kKeepBytes / tile_bytes;
        // (not when the second sweep writes a lot: with k = 2^24 and 2^27 of 2^28 the kept tail made the call
        // 3 % and 7 % slower instead of 4 % faster)
        const bool small_output = (size_t)k * (size_t)(eb + 8) <= ((size_t)32 << 20);
        if (batch == 1 && !row_offsets && small_output && row_tiles > keep_tiles) P.keep_from_tile = (u32)(row_tiles - keep_tiles);
    }
    P.seed = seed;
    for (int i = 0; i < c.npass; ++i) P.pass[i] = c.pass[i];

    hipStream_t st = (hipStream_t)hip_stream;
    ListPlan list;
    const bool by_list = make_list_plan(batch, n, k, dt, tuning, row_offsets != nullptr, (flags & RTOPK_FLAG_SORTED) != 0, &list);
    (void)hipGetLastError();  // an error left by earlier HIP calls of the process is not this call's
    const bool scaled = (flags & RTOPK_FLAG_SCALING) && dt == RTOPK_F32;
    if (by_list) {
        switch (dt) {
            case RTOPK_F32: return launch_list_f32(P, list, st, events);
            case RTOPK_F16: return launch_list_f16(P, list, st, events);
            case RTOPK_BF16: return launch_list_bf16(P, list, st, events);
        }
    }
    switch (dt) {
        case RTOPK_F32: return launch_f32(P, c, scaled, st, events);
        case RTOPK_F16: return launch_f16(P, c, false, st, events);
        case RTOPK_BF16: return launch_bf16(P, c, false, st, events);
    }
    return RTOPK_ERR_INVALID_ARG;
}

rtopk_status rtopk_select_events(const void* keys, int64_t batch, int64_t n, int64_t k, rtopk_dtype dt, int largest,
                                 uint32_t flags, uint64_t seed, void* out_values, int64_t* out_indices,
                                 void* workspace, size_t workspace_bytes, void* hip_stream,
                                 const rtopk_tuning* tuning, void* const* events) {
    return select_impl(keys, nullptr, nullptr, batch, n, k, dt, largest, flags, seed, out_values, out_indices, workspace,
                       workspace_bytes, hip_stream, tuning, events);
}

rtopk_status rtopk_select_ragged(const void* keys, const int64_t* row_offsets, const int64_t* row_k, int64_t batch,
                                 int64_t n_max, int64_t k_max, rtopk_dtype dt, int largest, uint32_t flags, uint64_t seed,
                                 void* out_values, int64_t* out_indices, void* workspace, size_t workspace_bytes,
                                 void* hip_stream, const rtopk_tuning* tuning) {
    if (!row_offsets || !row_k) return RTOPK_ERR_INVALID_ARG;
    if (((uintptr_t)row_offsets % 8) || ((uintptr_t)row_k % 8)) return RTOPK_ERR_UNSUPPORTED;
    return select_impl(keys, row_offsets, row_k, batch, n_max, k_max, dt, largest, flags, seed, out_values, out_indices,
                       workspace, workspace_bytes, hip_stream, tuning, nullptr);
}

rtopk_status rtopk_select_ex(const void* keys, int64_t batch, int64_t n, int64_t k, rtopk_dtype dt, int largest,
                             uint32_t flags, uint64_t seed, void* out_values, int64_t* out_indices, void* workspace,
                             size_t workspace_bytes, void* hip_stream, const rtopk_tuning* tuning) {
    return rtopk_select_events(keys, batch, n, k, dt, largest, flags, seed, out_values, out_indices, workspace,
                               workspace_bytes, hip_stream, tuning, nullptr);
}

rtopk_status rtopk_select(const void* keys, int64_t batch, int64_t n, int64_t k, rtopk_dtype dt, int largest,
                          uint32_t flags, uint64_t seed, void* out_values, int64_t* out_indices, void* workspace,
                          size_t workspace_bytes, void* hip_stream) {
    return rtopk_select_ex(keys, batch, n, k, dt, largest, flags, seed, out_values, out_indices, workspace,
                           workspace_bytes, hip_stream, nullptr);
}

rtopk_status rtopk_select_static(const void* keys, int64_t batch, int64_t n, int64_t k, rtopk_dtype dt, int largest,
                                 uint32_t flags, uint64_t seed, void* out_values, int64_t* out_indices,
                                 void* hip_stream) {
    size_t need = 0;
    const rtopk_status sized = rtopk_workspace_bytes(batch, n, k, dt, flags, &need);
    if (sized != RTOPK_OK) return sized;
    if (need > RTOPK_STATIC_SCRATCH_BYTES) return RTOPK_ERR_STATIC_SCRATCH;
    if (!keys || !out_values || !out_indices) return RTOPK_ERR_INVALID_ARG;
    void* ws = static_scratch_of_current_device();
    if (!ws) return RTOPK_ERR_HIP;
    // (every kernel chain starts by clearing the records, histograms and counters it relies on, so what the
    // previous call left in the buffer does not matter)
    return rtopk_select(keys, batch, n, k, dt, largest, flags, seed, out_values, out_indices, ws,
                        RTOPK_STATIC_SCRATCH_BYTES, hip_stream);
}

}  // extern "C"
