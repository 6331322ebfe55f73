// zk_batch_row_f64_5.hip -- batched row-pass kernel instances (double transforms);
// written by gen_batch_units.py.
#include "zk_kernels.hpp"

namespace zk {

extern const KernelEntry row_f64_5[];
const KernelEntry row_f64_5[] = {
    {2, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 2, 9, true>)},
    {2, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 2, 10, false>)},
    {8, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 8, 2, false>)},
    {8, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 8, 3, true>)},
    {8, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 8, 6, false>)},
    {16, 15, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 16, 15, true>)},
    {24, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 24, 3, true>)},
    {64, 3, true, KF_EARLY, reinterpret_cast<const void *>(&row_kernel_batch<double, 64, 3, true, false, true>)},
    {64, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 64, 6, true>)},
    {64, 9, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<double, 64, 9, true, true>)},
    {80, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 80, 2, false>)},
    {128, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 128, 3, true>)},
    {128, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 128, 4, false>)},
    {128, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 128, 10, false>)},
    {128, 12, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 128, 12, true>)},
    {256, 3, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<double, 256, 3, true, true>)},
    {384, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 384, 2, false>)},
    {384, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 384, 3, true>)},
    {0, 0, false, 0, nullptr}};

}  // namespace zk
