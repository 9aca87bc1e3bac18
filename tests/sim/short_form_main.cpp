// The short-form rescale of common.hpp (requant_short4), compiled for the host with stand-ins for its two
// instructions, against the 64-bit definition: every shift of its range, with and without a residual
// byte, both clamps, accumulators and multipliers at their extremes, around every step of the result
// and drawn at random.
#include "pw_pipe_sim_shim.hpp"

using namespace qasr;

namespace {

uint64_t state = 1;
uint32_t rnd32() {                                       // splitmix64
  uint64_t z = (state += 0x9e3779b97f4a7c15ull);
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  return (uint32_t)(z >> 32);
}

int64_t want(int32_t A, int32_t m, int s, int r, int lo) {
  const __int128 v = ((__int128)A * m + ((__int128)1 << (s - 1))) >> s;
  const __int128 w = v + r;
  return w < lo ? lo : w > 127 ? 127 : (int64_t)w;
}

long checked = 0;

template <bool RES, bool RELU>
void check(const int32_t (&A)[4], int32_t m, int s, const int (&r)[4]) {
  uint32_t rw = 0;
  for (int i = 0; i < 4; ++i) rw |= (uint32_t)(uint8_t)r[i] << (8 * i);
  const uint32_t got = requant_short4<RES, RELU>(A, m, s - 32, 1 << (s - 33), RES ? rw : 0u);
  for (int i = 0; i < 4; ++i) {
    const int64_t w = want(A[i], m, s, RES ? r[i] : 0, RELU ? 0 : -128);
    if ((int8_t)(got >> (8 * i)) != w) {
      std::printf("RES %d RELU %d: A %d m %d s %d residual %d: %d, not %d\n", RES, RELU, A[i], m, s, r[i],
                  (int)(int8_t)(got >> (8 * i)), (int)w);
      std::exit(1);
    }
    ++checked;
  }
}

template <bool RES>
void check_range(int s_max) {
  const int32_t ms[] = {0, 1, 1 << 30, (1 << 30) + 1, 0x7fffffff, 0x55555555};
  const int rs[] = {-128, -1, 0, 1, 127};
  for (int s = kShortMin; s <= s_max; ++s)
    for (int t = 0; t < 4000; ++t) {
      const int32_t m = t & 1 ? (int32_t)(rnd32() & 0x7fffffff) : ms[(t / 2) % 6];
      int32_t A[4];
      int r[4];
      for (int i = 0; i < 4; ++i) {
        const uint32_t k = rnd32();
        r[i] = k & 8 ? (int)(int8_t)rnd32() : rs[(k >> 4) % 5];
        if ((k & 3) == 0) A[i] = (int32_t)rnd32();
        else if ((k & 3) == 1) A[i] = k & 4 ? INT32_MAX - (int32_t)(k >> 28) : INT32_MIN + (int32_t)(k >> 28);
        else {                                           // near where the result steps to a value in -130 .. 130
          const int v = (int)(rnd32() % 261) - 130;
          const double a = m > 0 ? ((double)v - 0.5) * __builtin_ldexp(1.0, s) / m : 0.0;
          A[i] = (int32_t)std::max(-2147483648.0, std::min(2147483647.0, a + (double)((int)(rnd32() % 5) - 2)));
        }
      }
      check<RES, false>(A, m, s, r);
      check<RES, true>(A, m, s, r);
    }
}

}  // namespace

int main() {
  check_range<false>(kShortMax);
  check_range<true>(kShortMaxRes);
  std::printf("%ld values right\n", checked);
  return 0;
}
