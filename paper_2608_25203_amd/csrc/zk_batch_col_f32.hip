// zk_batch_col_f32.hip -- batched col-pass kernel instances (float transforms);
// written by gen_batch_units.py.
#include "zk_kernels.hpp"

namespace zk {

extern const KernelEntry col_f32_0[];
const KernelEntry col_f32_0[] = {
    {2, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 2, 2, false, false>)},
    {2, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 2, 3, false, true>)},
    {2, 4, false, KF_LIFTSYM, reinterpret_cast<const void *>(&col_kernel_batch<float, 2, 4, true, false>)},
    {2, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 2, 6, false, false>)},
    {2, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 2, 9, false, true>)},
    {2, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 2, 10, false, false>)},
    {2, 15, true, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 2, 15, false, true>)},
    {4, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 4, 2, false, false>)},
    {4, 4, false, KF_LIFTSYM, reinterpret_cast<const void *>(&col_kernel_batch<float, 4, 4, true, false>)},
    {4, 6, false, KF_LIFTSYM, reinterpret_cast<const void *>(&col_kernel_batch<float, 4, 6, true, false>)},
    {4, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 4, 6, false, true>)},
    {4, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 4, 10, false, false>)},
    {8, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 8, 2, false, false>)},
    {8, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 8, 3, false, true>)},
    {8, 4, false, KF_LIFTSYM, reinterpret_cast<const void *>(&col_kernel_batch<float, 8, 4, true, false>)},
    {8, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 8, 6, false, false>)},
    {8, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 8, 9, false, true>)},
    {8, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 8, 10, false, false>)},
    {8, 15, true, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 8, 15, false, true>)},
    {16, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 16, 2, false, false>)},
    {16, 4, false, KF_LIFTSYM, reinterpret_cast<const void *>(&col_kernel_batch<float, 16, 4, true, false>)},
    {16, 6, false, KF_LIFTSYM, reinterpret_cast<const void *>(&col_kernel_batch<float, 16, 6, true, false>)},
    {16, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 16, 6, false, true>)},
    {16, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 16, 10, false, false>)},
    {32, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 32, 2, false, false>)},
    {32, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 32, 3, false, true>)},
    {32, 4, false, KF_LIFTSYM, reinterpret_cast<const void *>(&col_kernel_batch<float, 32, 4, true, false>)},
    {32, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 32, 6, false, false>)},
    {32, 8, false, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 32, 8, false, false>)},
    {32, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 32, 9, false, true>)},
    {32, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 32, 10, false, false>)},
    {32, 15, true, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 32, 15, false, true>)},
    {64, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 64, 2, false, false>)},
    {64, 3, true, KF_FOLDS, reinterpret_cast<const void *>(&col_kernel_folds<float, 64, 3>)},
    {64, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 64, 4, false, false>)},
    {64, 6, false, KF_LIFTSYM, reinterpret_cast<const void *>(&col_kernel_batch<float, 64, 6, true, false>)},
    {64, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 64, 6, false, true>)},
    {64, 8, false, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 64, 8, false, false>)},
    {64, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 64, 10, false, false>)},
    {64, 12, true, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 64, 12, false, true>)},
    {128, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 128, 2, false, false>)},
    {128, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 128, 3, false, true>)},
    {128, 4, false, KF_LIFTSYM, reinterpret_cast<const void *>(&col_kernel_batch<float, 128, 4, true, false>)},
    {128, 6, false, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 128, 6, false, false>)},
    {128, 8, false, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 128, 8, false, false>)},
    {128, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 128, 9, false, true>)},
    {128, 10, false, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 128, 10, false, false>)},
    {128, 15, true, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 128, 15, false, true>)},
    {256, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 256, 2, false, false>)},
    {256, 3, true, KF_FOLDS, reinterpret_cast<const void *>(&col_kernel_folds<float, 256, 3>)},
    {256, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 256, 4, false, false>)},
    {256, 6, false, KF_LIFTSYM, reinterpret_cast<const void *>(&col_kernel_batch<float, 256, 6, true, false>)},
    {256, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 256, 6, false, true>)},
    {256, 9, true, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 256, 9, false, true>)},
    {512, 2, false, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 512, 2, false, false>)},
    {512, 3, true, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 512, 3, false, true>)},
    {512, 4, false, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 512, 4, false, false>)},
    {512, 6, true, KF_PLAIN, reinterpret_cast<const void *>(&col_kernel_batch<float, 512, 6, false, true>)},
    {0, 0, false, 0, nullptr}};

extern const KernelEntry col_f32_1[];
const KernelEntry *const col_kernels_f32[] = {col_f32_0, col_f32_1, nullptr};

}  // namespace zk
