// zk_batch_row_f32_3.hip -- batched row-pass kernel instances (float transforms);
// written by gen_batch_units.py.
#include "zk_kernels.hpp"

namespace zk {

extern const KernelEntry row_f32_3[];
const KernelEntry row_f32_3[] = {
    {4, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 4, 6, false>)},
    {8, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 8, 2, false>)},
    {8, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 8, 3, true>)},
    {8, 15, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 8, 15, true>)},
    {16, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 16, 6, true>)},
    {32, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 32, 3, true>)},
    {32, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 32, 4, false>)},
    {32, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 32, 9, true>)},
    {32, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 32, 10, false>)},
    {64, 8, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 64, 8, false>)},
    {64, 12, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 64, 12, true>)},
    {64, 15, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 64, 15, true>)},
    {128, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 128, 6, false>)},
    {128, 8, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 128, 8, false>)},
    {256, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 256, 2, false>)},
    {256, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 256, 6, true>)},
    {256, 8, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 256, 8, false>)},
    {256, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 256, 9, true>)},
    {1024, 3, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<float, 1024, 3, true, true>)},
    {0, 0, false, 0, nullptr}};

}  // namespace zk
