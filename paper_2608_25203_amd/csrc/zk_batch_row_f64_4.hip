// zk_batch_row_f64_4.hip -- batched row-pass kernel instances (double transforms);
// written by gen_batch_units.py.
#include "zk_kernels.hpp"

namespace zk {

extern const KernelEntry row_f64_4[];
const KernelEntry row_f64_4[] = {
    {2, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 2, 4, false>)},
    {8, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 8, 6, true>)},
    {32, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 32, 2, false>)},
    {32, 3, true, KF_EARLY, reinterpret_cast<const void *>(&row_kernel_batch<double, 32, 3, true, false, true>)},
    {32, 12, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 32, 12, true>)},
    {32, 15, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 32, 15, true>)},
    {64, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 64, 3, true>)},
    {64, 12, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<double, 64, 12, true, true>)},
    {128, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 128, 6, false>)},
    {128, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 128, 6, true>)},
    {128, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 128, 9, true>)},
    {160, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 160, 2, false>)},
    {256, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 256, 4, false>)},
    {256, 6, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<double, 256, 6, true, true>)},
    {256, 12, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 256, 12, true>)},
    {512, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 512, 3, true>)},
    {1024, 3, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<double, 1024, 3, true, true>)},
    {0, 0, false, 0, nullptr}};

}  // namespace zk
