// zk_batch_row_f64_1.hip -- batched row-pass kernel instances (double transforms);
// written by gen_batch_units.py.
#include "zk_kernels.hpp"

namespace zk {

extern const KernelEntry row_f64_1[];
const KernelEntry row_f64_1[] = {
    {2, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 2, 6, false>)},
    {4, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 4, 3, true>)},
    {4, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 4, 9, true>)},
    {16, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 16, 6, true>)},
    {40, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 40, 2, false>)},
    {64, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 64, 3, true>)},
    {64, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 64, 6, true>)},
    {64, 9, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<double, 64, 9, true, true>)},
    {64, 15, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 64, 15, true>)},
    {128, 12, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 128, 12, true>)},
    {192, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 192, 2, false>)},
    {256, 3, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<double, 256, 3, true, true>)},
    {256, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 256, 3, true>)},
    {256, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 256, 9, true>)},
    {768, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 768, 2, false>)},
    {768, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 768, 3, true>)},
    {0, 0, false, 0, nullptr}};

}  // namespace zk
