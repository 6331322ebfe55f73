// zk_launch.cpp -- lookup of the generated kernel instances by team shape.
#include <cstdint>

#include "zk_kernels.hpp"

namespace zk {

namespace {

uint32_t key_of(int row, int f64, int form, int T, int E, int pad) {
  return (uint32_t)(((((T * 16 + E) * 8 + form) * 2 + pad) * 2 + f64) * 2 + row);
}

// Hash table in static storage (a lookup runs inside every C entry point that
// launches, so building it must not allocate or throw); keys are never 0 (T > 0).
struct Table {
  static constexpr uint32_t kSlots = 4096;
  uint32_t key[kSlots] = {};
  const void *fn[kSlots] = {};
  static uint32_t slot(uint32_t k) { return (k * 2654435761u) >> 20; }
  Table() noexcept {
    const KernelEntry *const *const lists[2][2] = {{col_kernels_f32, col_kernels_f64},
                                                   {row_kernels_f32, row_kernels_f64}};
    uint32_t n = 0;
    for (int r = 0; r < 2; ++r)
      for (int d = 0; d < 2; ++d)
        for (const KernelEntry *const *l = lists[r][d]; *l; ++l)
          for (const KernelEntry *k = *l; k->T && n < kSlots / 2; ++k, ++n) {
            const uint32_t v = key_of(r, d, k->form, k->T, k->E, k->pad);
            uint32_t s = slot(v);
            while (key[s] && key[s] != v) s = (s + 1) % kSlots;
            key[s] = v;
            fn[s] = k->fn;
          }
  }
  const void *find(uint32_t v) const noexcept {
    uint32_t s = slot(v);
    while (key[s] && key[s] != v) s = (s + 1) % kSlots;
    return key[s] ? fn[s] : nullptr;
  }
};

}  // namespace

const void *find_kernel(bool row, bool f64, int form, int T, int E, bool pad) {
  static const Table table;
  return table.find(key_of(row, f64, form, T, E, pad));
}

}  // namespace zk
