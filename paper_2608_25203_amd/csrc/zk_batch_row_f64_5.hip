// zk_batch_row_f64_5.hip -- batched row-pass kernel instances (double transforms);
// written by gen_batch_units.py.
#include "zk_kernels.hpp"

namespace zk {

extern const KernelEntry row_f64_5[];
const KernelEntry row_f64_5[] = {
    {4, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 4, 4, false>)},
    {4, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 4, 6, true>)},
    {4, 15, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 4, 15, true>)},
    {8, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 8, 2, false>)},
    {8, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 8, 10, false>)},
    {16, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 16, 9, true>)},
    {24, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 24, 3, true>)},
    {32, 8, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 32, 8, false>)},
    {64, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 64, 4, false>)},
    {64, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 64, 10, false>)},
    {80, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 80, 2, false>)},
    {128, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 128, 3, true>)},
    {128, 6, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<double, 128, 6, true, true>)},
    {256, 9, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<double, 256, 9, true, true>)},
    {384, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 384, 2, false>)},
    {384, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 384, 3, true>)},
    {0, 0, false, 0, nullptr}};

}  // namespace zk
