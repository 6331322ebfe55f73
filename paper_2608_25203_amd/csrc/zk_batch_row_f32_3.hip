// zk_batch_row_f32_3.hip -- batched row-pass kernel instances (float transforms);
// written by gen_batch_units.py.
#include "zk_kernels.hpp"

namespace zk {

extern const KernelEntry row_f32_3[];
const KernelEntry row_f32_3[] = {
    {2, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 2, 4, false>)},
    {2, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 2, 9, true>)},
    {4, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 4, 2, false>)},
    {4, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 4, 6, false>)},
    {8, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 8, 10, false>)},
    {16, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 16, 6, true>)},
    {16, 15, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 16, 15, true>)},
    {32, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 32, 3, true>)},
    {64, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 64, 4, false>)},
    {64, 8, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 64, 8, false>)},
    {64, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 64, 9, true>)},
    {128, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 128, 2, false>)},
    {128, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 128, 6, false>)},
    {128, 8, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 128, 8, false>)},
    {128, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 128, 10, false>)},
    {128, 12, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 128, 12, true>)},
    {256, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 256, 6, true>)},
    {256, 8, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 256, 8, false>)},
    {0, 0, false, 0, nullptr}};

}  // namespace zk
