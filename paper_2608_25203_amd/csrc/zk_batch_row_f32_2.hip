// zk_batch_row_f32_2.hip -- batched row-pass kernel instances (float transforms);
// written by gen_batch_units.py.
#include "zk_kernels.hpp"

namespace zk {

extern const KernelEntry row_f32_2[];
const KernelEntry row_f32_2[] = {
    {2, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 2, 3, true>)},
    {2, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 2, 10, false>)},
    {4, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 4, 9, true>)},
    {8, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 8, 2, false>)},
    {8, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 8, 4, false>)},
    {8, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 8, 6, false>)},
    {32, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 32, 6, true>)},
    {32, 8, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 32, 8, false>)},
    {32, 12, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 32, 12, true>)},
    {32, 15, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 32, 15, true>)},
    {64, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 64, 3, true>)},
    {64, 12, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<float, 64, 12, true, true>)},
    {128, 12, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<float, 128, 12, true, true>)},
    {256, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 256, 4, false>)},
    {256, 12, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<float, 256, 12, true, true>)},
    {256, 12, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 256, 12, true>)},
    {512, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 512, 3, true>)},
    {512, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 512, 4, false>)},
    {0, 0, false, 0, nullptr}};

}  // namespace zk
