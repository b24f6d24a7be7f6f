// Host-side plan of one call: which kernels run, with what geometry.  Shared by the API translation
// unit and the per-type kernel translation units.
#pragma once
#include <hip/hip_runtime.h>
#include "rtopk.h"
#include "rtopk_device.h"

namespace rtopk {

struct Config {
    int d, path, G;
    int Gs;          // sorted output of long rows: workgroups per row of the radix sort (0: not needed)
    u32 small;
    int npass;
    bool one_sweep;  // path 1: try the one-sweep kernel (small k) first
    bool prefilter;  // path 2: histogram of a sample + ONE sweep over X that counts and filters, instead of two sweeps
    unsigned pre_stride;
    int multi_last;  // last digit pass that may still hold more than `small` candidates (grid kernels run up to it)
    u32 idx_max, dirmask;
    PassInfo pass[kMaxPasses];
};

// Enqueue every kernel of one call for one key type (defined in rtopk_f32.hip / rtopk_f16.hip / rtopk_bf16.hip).
rtopk_status launch_f32(const Params& P, const Config& c, bool scaled, hipStream_t st, void* const* events);
rtopk_status launch_f16(const Params& P, const Config& c, bool scaled, hipStream_t st, void* const* events);
rtopk_status launch_bf16(const Params& P, const Config& c, bool scaled, hipStream_t st, void* const* events);

// Plan of a call that goes through lists (rtopk_list.inl).  Offsets: bytes from the start of a row's working memory.
constexpr unsigned kListMaxBuckets = 4096;
constexpr unsigned kListSplits = 256;                  // intervals between splitters
constexpr int kListPartBlock = 256, kListPartVecs = 8;  // a stretch of a row that one workgroup holds: 32 KB
constexpr unsigned kListMetaBytes = 256;  // a row's records before the plan's first offset
// A bucket's places are taken from its beginning by every other workgroup, and from its end by the rest: two arrays of so many counters, not of the same cache line.  (k_list_emit counts two things
// in one.)
__host__ __device__ constexpr u32 list_cursors(u32 nb) { return (nb + 1u + 31u) & ~31u; }
struct ListPlan {
    int G;            // workgroups per row in the sweep
    int row_block;    // one workgroup per row does everything: its threads (0: many workgroups per row)
    int held;         // ... holding the row in registers: 16-byte vectors per thread (0: the row is swept)
    int sample;       // which size of sample: 512, 1024, 2048, 4096 or 16384 (16-bit keys, and 5: 8192) vectors of 16 bytes; k_list_stream's: 4096 and 8192 (4096)
    int stream_block; // short lists of few rows: threads of k_list_stream's workgroups, which take the sample themselves (0: k_list_bound does)
    int stream;       // the input is too large for the caches to keep: read past them
    int finish;       // short lists: threads of the workgroup that puts a row's list in order
    int ties;         // workgroups per row that fetch elements equal to the bound, where those are very many
    u32 seg_stride;   // the row's stretches are held by G workgroups that list at most this many each (0: the row is swept)
    u32 nb;           // long lists: buckets per row (0: short lists)
    int half;         // ... the sweep's tiles are of 32 KB, not of 64
    u32 hists;        // ... copies of the list's histogram
    u32 bucket_shift; // ... of 2^bucket_shift ranks
    u32 slots;        // short lists: a power of two: so many entries of each segment lie together at front_off
    u32 room, most;   // ... so many in all are put in order in LDS, longer ones are cut down first; the record says so from `most` on
    u32 front_off, hist_off, cursor_off, first_off, split_off, seg_off, tile_off, stack_off;
};
void launch_list_rows_f32(const Params& P, const ListPlan& L, hipStream_t st);  // (the kernels of L.row_block alone)
void launch_list_rows_f16(const Params& P, const ListPlan& L, hipStream_t st);
void launch_list_rows_bf16(const Params& P, const ListPlan& L, hipStream_t st);
rtopk_status launch_list_f32(const Params& P, const ListPlan& L, hipStream_t st, void* const* events);
rtopk_status launch_list_f16(const Params& P, const ListPlan& L, hipStream_t st, void* const* events);
rtopk_status launch_list_bf16(const Params& P, const ListPlan& L, hipStream_t st, void* const* events);

// Launch geometry the host needs for sizing.
constexpr int kHostHistBuffers = 6;  // global histograms per row: four in rotation, the sample's, the prefilter's second
constexpr int kHostSwgBuffers = 4;   // per-workgroup record sets per row: three in rotation, the prefilter's second
constexpr int kHostSortSmall = 8192;  // sorted output: rows of up to this many outputs are sorted by one workgroup in LDS
constexpr int kHostGridBlock = 512;
constexpr int kHostElemsPerLane = 16;

}  // namespace rtopk
