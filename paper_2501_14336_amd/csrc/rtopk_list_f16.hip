// List kernels for RTOPK_F16 keys.
#include "rtopk_list.inl"

namespace rtopk {
rtopk_status launch_list_f16(const Params& P, const ListPlan& L, hipStream_t st, void* const* events) {
    return launch_list_all<RTOPK_F16>(P, L, st, events, launch_list_rows_f16);
}
}  // namespace rtopk
