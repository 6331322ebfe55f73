// zk_batch_row_f64_6.hip -- batched row-pass kernel instances (double transforms);
// written by gen_batch_units.py.
#include "zk_kernels.hpp"

namespace zk {

extern const KernelEntry row_f64_6[];
const KernelEntry row_f64_6[] = {
    {4, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 4, 2, false>)},
    {4, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 4, 4, false>)},
    {4, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 4, 9, true>)},
    {8, 15, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 8, 15, true>)},
    {16, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 16, 6, false>)},
    {24, 3, true, KF_EARLY, reinterpret_cast<const void *>(&row_kernel_batch<double, 24, 3, true, false, true>)},
    {48, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 48, 3, true>)},
    {64, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 64, 2, false>)},
    {64, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 64, 10, false>)},
    {64, 12, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 64, 12, true>)},
    {128, 3, true, KF_EARLY, reinterpret_cast<const void *>(&row_kernel_batch<double, 128, 3, true, false, true>)},
    {128, 3, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<double, 128, 3, true, true>)},
    {256, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 256, 6, false>)},
    {256, 8, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 256, 8, false>)},
    {256, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 256, 9, true>)},
    {320, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 320, 2, false>)},
    {320, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 320, 3, true>)},
    {512, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 512, 4, false>)},
    {0, 0, false, 0, nullptr}};

}  // namespace zk
