// zk_batch_row_f64_2.hip -- batched row-pass kernel instances (double transforms);
// written by gen_batch_units.py.
#include "zk_kernels.hpp"

namespace zk {

extern const KernelEntry row_f64_2[];
const KernelEntry row_f64_2[] = {
    {2, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 2, 6, true>)},
    {4, 15, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 4, 15, true>)},
    {8, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 8, 10, false>)},
    {16, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 16, 4, false>)},
    {16, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 16, 9, true>)},
    {24, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 24, 2, false>)},
    {32, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 32, 6, false>)},
    {40, 3, true, KF_EARLY, reinterpret_cast<const void *>(&row_kernel_batch<double, 40, 3, true, false, true>)},
    {64, 3, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<double, 64, 3, true, true>)},
    {80, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 80, 3, true>)},
    {128, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 128, 2, false>)},
    {128, 8, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 128, 8, false>)},
    {128, 15, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 128, 15, true>)},
    {192, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 192, 3, true>)},
    {256, 12, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<double, 256, 12, true, true>)},
    {640, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 640, 2, false>)},
    {640, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 640, 3, true>)},
    {1024, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 1024, 2, false>)},
    {0, 0, false, 0, nullptr}};

}  // namespace zk
