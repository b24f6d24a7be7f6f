// List kernels for RTOPK_F32 keys.
#include "rtopk_list.inl"

namespace rtopk {
rtopk_status launch_list_f32(const Params& P, const ListPlan& L, hipStream_t st, void* const* events) {
    return launch_list_all<RTOPK_F32>(P, L, st, events, launch_list_rows_f32);
}
}  // namespace rtopk
