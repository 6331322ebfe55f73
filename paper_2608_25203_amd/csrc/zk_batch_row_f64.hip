// zk_batch_row_f64.hip -- batched row-pass kernel instances (double transforms);
// written by gen_batch_units.py.
#include "zk_kernels.hpp"

namespace zk {

extern const KernelEntry row_f64_0[];
const KernelEntry row_f64_0[] = {
    {2, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 2, 2, false>)},
    {4, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 4, 3, true>)},
    {4, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 4, 6, true>)},
    {16, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 16, 3, true>)},
    {32, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 32, 10, false>)},
    {48, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 48, 2, false>)},
    {48, 3, true, KF_EARLY, reinterpret_cast<const void *>(&row_kernel_batch<double, 48, 3, true, false, true>)},
    {64, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 64, 4, false>)},
    {64, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 64, 6, false>)},
    {64, 8, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 64, 8, false>)},
    {64, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 64, 9, true>)},
    {96, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 96, 3, true>)},
    {128, 12, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<double, 128, 12, true, true>)},
    {256, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 256, 2, false>)},
    {256, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 256, 6, true>)},
    {512, 6, true, KF_LANES, reinterpret_cast<const void *>(&row_kernel_batch<double, 512, 6, true, true>)},
    {1024, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&row_kernel_batch<double, 1024, 3, true>)},
    {0, 0, false, 0, nullptr}};

extern const KernelEntry row_f64_1[];
extern const KernelEntry row_f64_2[];
extern const KernelEntry row_f64_3[];
extern const KernelEntry row_f64_4[];
extern const KernelEntry row_f64_5[];
extern const KernelEntry row_f64_6[];
const KernelEntry *const row_kernels_f64[] = {row_f64_0, row_f64_1, row_f64_2, row_f64_3, row_f64_4, row_f64_5, row_f64_6, nullptr};

}  // namespace zk
