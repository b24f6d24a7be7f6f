// List kernels of rows that one workgroup takes alone, for RTOPK_F16 keys.
#include "rtopk_list.inl"

namespace rtopk {
void launch_list_rows_f16(const Params& P, const ListPlan& L, hipStream_t st) { launch_rows<RTOPK_F16>(P, L, st); }
}  // namespace rtopk
