// zk_batch_row_f32_1.hip -- batched row-pass kernel instances (float transforms);
// written by gen_batch_units.py.
#include "zk_kernels.hpp"

namespace zk {

extern const KernelEntry row_f32_1[];
const KernelEntry row_f32_1[] = {
    {2, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 2, 6, false>)},
    {2, 15, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 2, 15, true>)},
    {4, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 4, 3, true>)},
    {8, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 8, 6, true>)},
    {8, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 8, 9, true>)},
    {16, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 16, 2, false>)},
    {16, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 16, 4, false>)},
    {16, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 16, 10, false>)},
    {64, 3, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<float, 64, 3, true, true>)},
    {64, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 64, 6, false>)},
    {64, 15, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 64, 15, true>)},
    {128, 3, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<float, 128, 3, true, true>)},
    {128, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 128, 3, true>)},
    {128, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 128, 9, true>)},
    {256, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 256, 2, false>)},
    {256, 3, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<float, 256, 3, true, true>)},
    {512, 3, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<float, 512, 3, true, true>)},
    {512, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 512, 6, true>)},
    {0, 0, false, 0, nullptr}};

}  // namespace zk
