// zk_batch_row_f32_1.hip -- batched row-pass kernel instances (float transforms);
// written by gen_batch_units.py.
#include "zk_kernels.hpp"

namespace zk {

extern const KernelEntry row_f32_1[];
const KernelEntry row_f32_1[] = {
    {4, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 4, 4, false>)},
    {4, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 4, 10, false>)},
    {8, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 8, 6, false>)},
    {8, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 8, 9, true>)},
    {16, 3, true, KF_EARLY, reinterpret_cast<const void *>(&row_kernel_batch<float, 16, 3, true, false, true>)},
    {32, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 32, 2, false>)},
    {32, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 32, 6, true>)},
    {64, 3, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<float, 64, 3, true, true>)},
    {128, 3, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<float, 128, 3, true, true>)},
    {128, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 128, 3, true>)},
    {128, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 128, 4, false>)},
    {128, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 128, 10, false>)},
    {256, 3, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<float, 256, 3, true, true>)},
    {256, 12, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 256, 12, true>)},
    {512, 3, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<float, 512, 3, true, true>)},
    {512, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 512, 4, false>)},
    {512, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 512, 6, true>)},
    {1024, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 1024, 2, false>)},
    {0, 0, false, 0, nullptr}};

}  // namespace zk
