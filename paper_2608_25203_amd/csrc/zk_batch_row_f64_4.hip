// zk_batch_row_f64_4.hip -- batched row-pass kernel instances (double transforms);
// written by gen_batch_units.py.
#include "zk_kernels.hpp"

namespace zk {

extern const KernelEntry row_f64_4[];
const KernelEntry row_f64_4[] = {
    {8, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 8, 4, false>)},
    {8, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 8, 6, false>)},
    {8, 15, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 8, 15, true>)},
    {16, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 16, 2, false>)},
    {16, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 16, 10, false>)},
    {32, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 32, 3, true>)},
    {32, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 32, 9, true>)},
    {64, 3, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<double, 64, 3, true, true>)},
    {96, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 96, 2, false>)},
    {128, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 128, 4, false>)},
    {128, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 128, 6, true>)},
    {128, 8, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 128, 8, false>)},
    {128, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 128, 10, false>)},
    {256, 12, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<double, 256, 12, true, true>)},
    {512, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 512, 2, false>)},
    {512, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 512, 3, true>)},
    {0, 0, false, 0, nullptr}};

}  // namespace zk
