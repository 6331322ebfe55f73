// zk_batch_row_f32_2.hip -- batched row-pass kernel instances (float transforms);
// written by gen_batch_units.py.
#include "zk_kernels.hpp"

namespace zk {

extern const KernelEntry row_f32_2[];
const KernelEntry row_f32_2[] = {
    {2, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 2, 4, false>)},
    {2, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 2, 10, false>)},
    {4, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 4, 6, true>)},
    {4, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 4, 9, true>)},
    {16, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 16, 2, false>)},
    {16, 15, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 16, 15, true>)},
    {32, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 32, 6, false>)},
    {32, 8, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 32, 8, false>)},
    {64, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 64, 3, true>)},
    {64, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 64, 4, false>)},
    {64, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 64, 10, false>)},
    {64, 12, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<float, 64, 12, true, true>)},
    {128, 12, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<float, 128, 12, true, true>)},
    {128, 12, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 128, 12, true>)},
    {128, 15, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 128, 15, true>)},
    {256, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 256, 4, false>)},
    {256, 12, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<float, 256, 12, true, true>)},
    {512, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 512, 2, false>)},
    {512, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 512, 3, true>)},
    {0, 0, false, 0, nullptr}};

}  // namespace zk
