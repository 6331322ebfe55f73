// zk_batch_row_f64_3.hip -- batched row-pass kernel instances (double transforms);
// written by gen_batch_units.py.
#include "zk_kernels.hpp"

namespace zk {

extern const KernelEntry row_f64_3[];
const KernelEntry row_f64_3[] = {
    {8, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 8, 6, true>)},
    {16, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 16, 4, false>)},
    {16, 15, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 16, 15, true>)},
    {24, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 24, 2, false>)},
    {32, 12, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 32, 12, true>)},
    {40, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 40, 3, true>)},
    {64, 6, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<double, 64, 6, true, true>)},
    {64, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 64, 9, true>)},
    {128, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 128, 2, false>)},
    {128, 9, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<double, 128, 9, true, true>)},
    {160, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 160, 3, true>)},
    {256, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 256, 4, false>)},
    {512, 3, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<double, 512, 3, true, true>)},
    {512, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 512, 6, true>)},
    {640, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 640, 2, false>)},
    {1024, 3, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<double, 1024, 3, true, true>)},
    {0, 0, false, 0, nullptr}};

}  // namespace zk
