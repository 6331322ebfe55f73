// zk_batch_row_f32.hip -- batched row-pass kernel instances (float transforms);
// written by gen_batch_units.py.
#include "zk_kernels.hpp"

namespace zk {

extern const KernelEntry row_f32_0[];
const KernelEntry row_f32_0[] = {
    {2, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 2, 2, false>)},
    {2, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 2, 3, true>)},
    {2, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 2, 6, false>)},
    {2, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 2, 9, true>)},
    {2, 15, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 2, 15, true>)},
    {8, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 8, 4, false>)},
    {8, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 8, 6, true>)},
    {8, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 8, 10, false>)},
    {16, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 16, 3, true>)},
    {64, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 64, 2, false>)},
    {64, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 64, 6, false>)},
    {64, 9, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<float, 64, 9, true, true>)},
    {64, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 64, 9, true>)},
    {128, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 128, 6, true>)},
    {128, 9, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<float, 128, 9, true, true>)},
    {256, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 256, 6, false>)},
    {256, 9, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<float, 256, 9, true, true>)},
    {1024, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<float, 1024, 3, true>)},
    {0, 0, false, 0, nullptr}};

extern const KernelEntry row_f32_1[];
extern const KernelEntry row_f32_2[];
extern const KernelEntry row_f32_3[];
extern const KernelEntry row_f32_4[];
const KernelEntry *const row_kernels_f32[] = {row_f32_0, row_f32_1, row_f32_2, row_f32_3, row_f32_4, nullptr};

}  // namespace zk
