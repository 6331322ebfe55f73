// zk_batch_row_f32_4.hip -- batched row-pass kernel instances (float transforms);
// written by gen_batch_units.py.
#include "zk_kernels.hpp"

namespace zk {

extern const KernelEntry row_f32_4[];
const KernelEntry row_f32_4[] = {
    {2, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 2, 6, true>)},
    {4, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 4, 2, false>)},
    {4, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 4, 3, true>)},
    {4, 15, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 4, 15, true>)},
    {16, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 16, 4, false>)},
    {16, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 16, 6, false>)},
    {16, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 16, 9, true>)},
    {16, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 16, 10, false>)},
    {32, 3, true, KF_EARLY, reinterpret_cast<const void *>(&row_kernel_batch<float, 32, 3, true, false, true>)},
    {32, 12, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 32, 12, true>)},
    {32, 15, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 32, 15, true>)},
    {64, 6, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<float, 64, 6, true, true>)},
    {64, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 64, 6, true>)},
    {128, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 128, 2, false>)},
    {128, 6, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<float, 128, 6, true, true>)},
    {128, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 128, 9, true>)},
    {256, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 256, 3, true>)},
    {256, 6, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<float, 256, 6, true, true>)},
    {512, 6, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<float, 512, 6, true, true>)},
    {0, 0, false, 0, nullptr}};

}  // namespace zk
