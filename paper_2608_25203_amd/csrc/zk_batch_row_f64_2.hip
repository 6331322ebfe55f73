// zk_batch_row_f64_2.hip -- batched row-pass kernel instances (double transforms);
// written by gen_batch_units.py.
#include "zk_kernels.hpp"

namespace zk {

extern const KernelEntry row_f64_2[];
const KernelEntry row_f64_2[] = {
    {2, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 2, 3, true>)},
    {2, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 2, 9, true>)},
    {16, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 16, 6, false>)},
    {32, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 32, 2, false>)},
    {32, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 32, 4, false>)},
    {32, 15, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 32, 15, true>)},
    {48, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 48, 3, true>)},
    {64, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 64, 6, false>)},
    {64, 8, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 64, 8, false>)},
    {64, 12, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 64, 12, true>)},
    {128, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 128, 9, true>)},
    {128, 12, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<double, 128, 12, true, true>)},
    {160, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 160, 2, false>)},
    {192, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 192, 3, true>)},
    {512, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 512, 4, false>)},
    {640, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 640, 3, true>)},
    {0, 0, false, 0, nullptr}};

}  // namespace zk
