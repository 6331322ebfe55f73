// zk_launch.cpp -- lookup of the generated kernel instances by team shape.
#include <cstdint>
#include <unordered_map>

#include "zk_kernels.hpp"

namespace zk {

const void *find_kernel(bool row, bool f64, int form, int T, int E, bool pad) {
  auto key = [](int r, int d, int f, int t, int e, int p) {
    return (uint32_t)(((((t * 16 + e) * 8 + f) * 2 + p) * 2 + d) * 2 + r);
  };
  static const std::unordered_map<uint32_t, const void *> table = [&] {
    std::unordered_map<uint32_t, const void *> m;
    const KernelEntry *const *const lists[2][2] = {{col_kernels_f32, col_kernels_f64},
                                                   {row_kernels_f32, row_kernels_f64}};
    for (int r = 0; r < 2; ++r)
      for (int d = 0; d < 2; ++d)
        for (const KernelEntry *const *l = lists[r][d]; *l; ++l)
          for (const KernelEntry *k = *l; k->T; ++k) m[key(r, d, k->form, k->T, k->E, k->pad)] = k->fn;
    return m;
  }();
  const auto it = table.find(key(row, f64, form, T, E, pad));
  return it == table.end() ? nullptr : it->second;
}

}  // namespace zk
