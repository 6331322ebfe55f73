// zk_batch_row_f64_3.hip -- batched row-pass kernel instances (double transforms);
// written by gen_batch_units.py.
#include "zk_kernels.hpp"

namespace zk {

extern const KernelEntry row_f64_3[];
const KernelEntry row_f64_3[] = {
    {2, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 2, 6, false>)},
    {2, 15, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 2, 15, true>)},
    {4, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 4, 10, false>)},
    {8, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 8, 4, false>)},
    {8, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 8, 9, true>)},
    {16, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 16, 2, false>)},
    {16, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 16, 6, true>)},
    {32, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 32, 3, true>)},
    {32, 8, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 32, 8, false>)},
    {64, 15, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 64, 15, true>)},
    {80, 3, true, KF_EARLY, reinterpret_cast<const void *>(&row_kernel_batch<double, 80, 3, true, false, true>)},
    {96, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 96, 2, false>)},
    {128, 6, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<double, 128, 6, true, true>)},
    {160, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 160, 3, true>)},
    {256, 9, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<double, 256, 9, true, true>)},
    {512, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 512, 2, false>)},
    {512, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 512, 6, true>)},
    {768, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 768, 2, false>)},
    {0, 0, false, 0, nullptr}};

}  // namespace zk
