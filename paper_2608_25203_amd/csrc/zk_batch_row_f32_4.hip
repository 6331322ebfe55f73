// zk_batch_row_f32_4.hip -- batched row-pass kernel instances (float transforms);
// written by gen_batch_units.py.
#include "zk_kernels.hpp"

namespace zk {

extern const KernelEntry row_f32_4[];
const KernelEntry row_f32_4[] = {
    {2, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 2, 2, false>)},
    {4, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 4, 4, false>)},
    {4, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 4, 6, true>)},
    {4, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 4, 10, false>)},
    {8, 15, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 8, 15, true>)},
    {16, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 16, 3, true>)},
    {32, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 32, 6, false>)},
    {32, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 32, 9, true>)},
    {64, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 64, 2, false>)},
    {64, 9, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<float, 64, 9, true, true>)},
    {64, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 64, 10, false>)},
    {64, 12, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 64, 12, true>)},
    {128, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 128, 4, false>)},
    {128, 9, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<float, 128, 9, true, true>)},
    {256, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 256, 3, true>)},
    {256, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 256, 6, false>)},
    {256, 9, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<float, 256, 9, true, true>)},
    {1024, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 1024, 2, false>)},
    {1024, 3, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<float, 1024, 3, true, true>)},
    {0, 0, false, 0, nullptr}};

}  // namespace zk
