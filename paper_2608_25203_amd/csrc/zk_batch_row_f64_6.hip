// zk_batch_row_f64_6.hip -- batched row-pass kernel instances (double transforms);
// written by gen_batch_units.py.
#include "zk_kernels.hpp"

namespace zk {

extern const KernelEntry row_f64_6[];
const KernelEntry row_f64_6[] = {
    {2, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 2, 4, false>)},
    {2, 15, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 2, 15, true>)},
    {4, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 4, 2, false>)},
    {4, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 4, 6, false>)},
    {4, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 4, 10, false>)},
    {8, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 8, 9, true>)},
    {16, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 16, 3, true>)},
    {32, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 32, 6, true>)},
    {32, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 32, 10, false>)},
    {64, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 64, 2, false>)},
    {96, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 96, 3, true>)},
    {128, 3, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<double, 128, 3, true, true>)},
    {256, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 256, 6, false>)},
    {256, 8, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 256, 8, false>)},
    {320, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 320, 2, false>)},
    {320, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 320, 3, true>)},
    {0, 0, false, 0, nullptr}};

}  // namespace zk
