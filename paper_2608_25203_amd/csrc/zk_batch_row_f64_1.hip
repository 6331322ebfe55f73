// zk_batch_row_f64_1.hip -- batched row-pass kernel instances (double transforms);
// written by gen_batch_units.py.
#include "zk_kernels.hpp"

namespace zk {

extern const KernelEntry row_f64_1[];
const KernelEntry row_f64_1[] = {
    {2, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 2, 3, true>)},
    {4, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 4, 6, false>)},
    {16, 3, true, KF_EARLY, reinterpret_cast<const void *>(&row_kernel_batch<double, 16, 3, true, false, true>)},
    {16, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 16, 10, false>)},
    {32, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 32, 4, false>)},
    {32, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 32, 6, true>)},
    {32, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 32, 9, true>)},
    {40, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 40, 2, false>)},
    {40, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 40, 3, true>)},
    {64, 6, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<double, 64, 6, true, true>)},
    {96, 3, true, KF_EARLY, reinterpret_cast<const void *>(&row_kernel_batch<double, 96, 3, true, false, true>)},
    {128, 9, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<double, 128, 9, true, true>)},
    {192, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 192, 2, false>)},
    {256, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 256, 3, true>)},
    {512, 3, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<double, 512, 3, true, true>)},
    {768, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 768, 3, true>)},
    {0, 0, false, 0, nullptr}};

}  // namespace zk
