// How many workgroups a launch may ask for: a grid is refused if one of its dimensions has 2^32 work items.
#pragma once
#include <stdint.h>

namespace qasr {

// the most workgroups of a launch along one dimension that is rounded up to a multiple of 8 (one run per XCD)
constexpr int64_t max_workgroups(int threads) { return (0xffffffffll / threads) & ~7ll; }

// A workgroup (of up to 1024 threads) per unit of work, in two dimensions beyond 2^20 of them: workgroup (x, y) takes
// unit y 2^20 + x, those past the last unit do nothing.
constexpr int kGridShift = 20;
struct GridShape { uint32_t x, y; };
constexpr GridShape grid_shape(int64_t units) {
  return units <= (1ll << kGridShift)
             ? GridShape{(uint32_t)units, 1u}
             : GridShape{1u << kGridShift, (uint32_t)((units + (1ll << kGridShift) - 1) >> kGridShift)};
}

}  // namespace qasr
