// CPU replay of the request bookkeeping of the dense kernels (csrc/conv_pipe.hip, csrc/conv_few.hip), in the manner of
// dw_pipe_sim_main.cpp: source and launcher are compiled for the host (conv_few with -DSIM_FEW) against pw_pipe_sim_shim.hpp, a launch runs
// every lane of every workgroup, the lanes' records are merged per wave and replayed under in-order completion
// with the latest completion the waits allow.  Checked:
//   * every global address lies inside its operand, every LDS address inside the launch's dynamic LDS;
//   * the lanes of a wave agree on wait counts, barriers, uniform values and stores;
//   * every register that a request fills is complete when it is tied, and every one is tied;
//   * no request into LDS is outstanding at a barrier, nothing is outstanding when a wave ends;
//   * no 16 bytes of LDS are written by one wave and read or written by another between the same two barriers;
//   * every output byte is written exactly once (pad bytes between rows at most once);
//   * conv_few asks ahead for the lines of the next layer's weights that the same die will read, once each.
#include "pw_pipe_sim_shim.hpp"

#include <atomic>
#include <cmath>
#include <functional>
#include <map>
#include <set>
#include <type_traits>

// ---- host side of a launch
typedef int hipError_t;
typedef void* hipStream_t;
constexpr int hipSuccess = 0, hipErrorInvalidValue = 1;
struct dim3 {
  unsigned x, y, z;
  dim3(unsigned a, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
#define __builtin_amdgcn_fence(order, scope) ((void)0)
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_fetch_add(p, v, order, scope) ((void)(p), qasr::sim_arrival())
#define __hip_atomic_store(p, v, order, scope) ((void)(p))
#define __builtin_amdgcn_raw_buffer_load_b128(r, off, soff, aux) sim_buffer_load16(r, (uint32_t)(off) + (uint32_t)(soff))
typedef unsigned sim_v4u __attribute__((ext_vector_type(4)));
inline sim_v4u sim_buffer_load16(SimRsrc r, uint32_t off) {
  if ((uint64_t)off + 16 > r.num) sim::fail("buffer load beyond the resource's size");
  sim::region_of(r.p + off, 16, false);
  return (sim_v4u){0, 0, 0, 0};
}

namespace qasr {

struct Tuning {
  bool no_conv_pipe = false, no_conv_few = false, conv_few_force = false, cp_plain_order = false;
  int cp_mt = 0, cp_nt = 0, cp_kg = 0, cp_s = 0, cf_mt = 0, cf_wc = 0, cf_nt = 0;
};
inline Tuning& the_tuning() { static Tuning t; return t; }
inline int g_tuning_asked = 0;                   // (every choice of a tile asks)
inline const Tuning& tuning() { ++g_tuning_asked; return the_tuning(); }
struct FewTile { int MT, WC, NT; };

inline int32_t dyadic_rescale(int32_t A, int32_t m, int32_t s) { return dyadic_rescale64(A, m, std::max(1, std::min(62, s))); }
inline int32_t clamp_i8(int32_t v, int32_t lo) { return std::min(127, std::max(lo, v)); }
inline uint32_t load_u32(const int8_t* p) { sim::region_of(p, 4, false); return 0; }
inline void store_row_u32(int8_t* row, int t, int T, uint32_t) {
  sim::count_store(row + t, (size_t)std::min(4, T - t));
}
constexpr int kMaxMoreRes = 11, kConvSplitCounters = 1024;

inline hipError_t ensure_max_dynamic_lds(const void*, std::atomic<uint64_t>&) { return hipSuccess; }
void run_launch(const std::function<void()>& lane, unsigned grid, unsigned threads, size_t lds);
template <typename G>
hipError_t launch_kernel(void (*kernel)(ConvParams, G), dim3 grid, dim3 block, size_t shmem, hipStream_t, ConvParams p, G g) {
  run_launch([=] { kernel(p, g); }, grid.x, block.x, shmem);
  return hipSuccess;
}
inline hipError_t launch_kernel(void (*)(unsigned*), dim3, dim3, size_t, hipStream_t, unsigned*) { return hipSuccess; }
// what thread 0 of the workgroup at hand is told when it counts its arrival: the last one finishes the tile
inline unsigned g_arrival = 0;
inline unsigned sim_arrival() { return g_arrival; }

}  // namespace qasr

#include "divide_extract.hpp"
#ifdef SIM_FEW
#include "conv_few_stripped.hpp"
#else
namespace qasr { inline bool conv_few_cycles(const ConvParams&, FewTile&, double&) { return false; } }
#include "conv_pipe_stripped.hpp"
#endif

namespace {

using namespace qasr;

struct Req { sim::Kind k; bool done; };

void replay(const std::vector<sim::Ev>& ev) {
  std::vector<Req> reqs;
  size_t head = 0;
  std::map<int64_t, size_t> reg_req;
  std::set<int64_t> tied;
  for (const sim::Ev& e : ev) {
    switch (e.k) {
      case sim::ISSUE_LDS: reqs.push_back(Req{e.k, false}); break;
      case sim::ISSUE_REG: reg_req[e.a] = reqs.size(); reqs.push_back(Req{e.k, false}); break;
      case sim::STORE: reqs.push_back(Req{e.k, false}); break;
      case sim::WAIT:
        if (e.b < 0) sim::fail("a run-time wait count is negative");
        while (reqs.size() - head > (size_t)e.a) reqs[head++].done = true;
        break;
      case sim::USE_REG: {
        auto it = reg_req.find(e.a);
        if (it == reg_req.end()) sim::fail("tie of a register no load was issued for");
        if (!reqs[it->second].done) sim::fail("a register is used before its load has completed");
        tied.insert(e.a);
        break;
      }
      case sim::BARRIER:
        for (const Req& r : reqs)
          if (r.k == sim::ISSUE_LDS && !r.done) sim::fail("a load into LDS is outstanding at a barrier");
        break;
      default: break;
    }
  }
  if (head != reqs.size()) sim::fail("requests are outstanding when the wave ends");
  if (tied.size() != reg_req.size()) sim::fail("a register that a load fills is never tied");
}

// 16-byte blocks of LDS by barrier interval: the waves that write and read them (a wave's own order is its program's)
struct Blocks {
  std::map<std::pair<int, int64_t>, std::pair<uint32_t, uint32_t>> at;
  void add(int wave, const std::vector<sim::Ev>& ev) {
    int interval = 0;
    for (const sim::Ev& e : ev) {
      if (e.k == sim::BARRIER) ++interval;
      if (e.k != sim::USE_LDS && e.k != sim::LDS_WRITE) continue;
      for (int64_t b : {e.a / 16, (e.a + 15) / 16}) (e.k == sim::LDS_WRITE ? at[{interval, b}].first : at[{interval, b}].second) |= 1u << wave;
    }
  }
  void check() const {
    for (const auto& [key, use] : at) {
      const uint32_t w = use.first, all = w | use.second;
      if (w && (all & (all - 1))) sim::fail("LDS block " + std::to_string(key.second) + " is shared between waves without a barrier");
    }
  }
};

long g_workgroups = 0;
std::string g_name;

}  // namespace

void qasr::run_launch(const std::function<void()>& lane, unsigned grid, unsigned threads, size_t lds_size) {
  auto& st = sim::S();
  for (unsigned wg = 0; wg < grid; ++wg) {
    std::vector<unsigned char> lds(lds_size, 0);
    st.lds = lds.data(); st.lds_bytes = lds_size;
    blockIdx.x = wg;
    st.where = g_name + " workgroup " + std::to_string(wg);
    Blocks blocks;
    for (unsigned wv = 0; wv < threads / 64; ++wv) {
      sim::Wave w;
      w.lanes.resize(64);
      for (int l = 0; l < 64; ++l) {
        st.ev.clear(); st.lane = l; st.wave = (int)wv; st.next_uid = 1;
        threadIdx.x = wv * 64 + (unsigned)l;
        lane();
        w.lanes[l] = st.ev;
        blocks.add((int)wv, st.ev);
      }
      st.lane = -1;
      replay(sim::merge(w));
    }
    blocks.check();
    ++g_workgroups;
  }
}

namespace {

struct Case {
  const char* name;
  int few, a, b, kg, s;            // conv_few: MT, WC, NT (0: 2); conv_pipe: MT, NT, groups, splits
  int B, Cin, Cout, T, k, stride, dil, pl, pr, res, bias, pad;
};

#ifdef SIM_FEW
// A workgroup's die is its number modulo 8; a launch gives die x the x-th of eight equal runs of its tiles, channel tile first.
int tiles_of(const ConvParams& p, const FewTile& t, int die, int& first) {
  const int bt = p.B * ((p.Tout + 16 * t.MT - 1) / (16 * t.MT)), ch = 16 * t.WC * t.NT, tiles = bt * ((p.Cout + ch - 1) / ch), run = (tiles + 7) / 8;
  first = die * run;
  return std::max(0, std::min(run, tiles - first));
}

// Whether the workgroups of each die have asked, once each, for the lines that the next layer's workgroups on that die will read: all
// of them, or from the first on as many as there are lanes (idle lanes ask for the first line of the weights).
void check_lines(const ConvParams& p, const FewTile& tile, const ConvParams& next, const FewTile& next_tile, size_t bytes) {
  const int bt = next.B * ((next.Tout + 16 * next_tile.MT - 1) / (16 * next_tile.MT)), columns = (next.Cout + 15) / 16, chunks = next.Cin / 64;
  for (int die = 0; die < 8; ++die) {
    int first = 0;
    const int lanes = tiles_of(p, tile, die, first) * 1024, n = tiles_of(next, next_tile, die, first);
    std::set<int64_t> reads;                        // lines of 128 bytes
    for (int v = first; v < first + n; ++v)
      for (int c = 0; c < next_tile.WC * next_tile.NT; ++c)
        for (int j = 0; j < next.k; ++j)
          for (int kc = 0; kc < chunks; ++kc)
            for (int l = 0; l < 8; ++l)
              if (v / bt * next_tile.WC * next_tile.NT + c < columns)
                reads.insert((((int64_t)j * columns + v / bt * next_tile.WC * next_tile.NT + c) * chunks + kc) * 8 + l);
    std::map<int64_t, int> asked;
    for (const auto& [wg, at] : sim::S().asked)
      if ((int)(wg & 7) == die && at >= (const unsigned char*)next.w && at < (const unsigned char*)next.w + bytes) ++asked[(at - (const unsigned char*)next.w) / 128];
    int64_t i = 0;
    for (int64_t line : reads) {
      const auto it = asked.find(line);
      if (i++ < lanes ? it == asked.end() || (line && it->second != 1) : line && it != asked.end())
        sim::fail("die " + std::to_string(die) + ": line " + std::to_string(line) + " is asked for " + std::to_string(it == asked.end() ? 0 : it->second) + " times");
    }
    for (const auto& [line, times] : asked)
      if (line && !reads.count(line)) sim::fail("die " + std::to_string(die) + " asks for line " + std::to_string(line) + ", which it does not read");
  }
}
#endif

void run_case(const Case& c) {
  Tuning& t = the_tuning();
  t = Tuning();
  if (c.few) { t.cf_mt = c.a; t.cf_wc = c.b; t.cf_nt = c.kg ? c.kg : 2; }
  else { t.cp_mt = c.a; t.cp_nt = c.b; t.cp_kg = c.kg; t.cp_s = c.s; }
  ConvParams p{};
  p.B = c.B; p.Cin = c.Cin; p.Cout = c.Cout; p.Tin = c.T; p.k = c.k; p.stride = c.stride; p.dil = c.dil; p.pl = c.pl;
  p.Tout = (c.T + c.pl + c.pr - c.dil * (c.k - 1) - 1) / c.stride + 1;
  p.xpad = c.pad ? (16 - p.Tin % 16) % 16 : 0; p.ypad = c.pad ? (16 - p.Tout % 16) % 16 : 0;
  p.xbs = (int64_t)p.Cin * (p.Tin + p.xpad); p.ybs = (int64_t)p.Cout * (p.Tout + p.ypad);
  p.relu = 1; p.w_packed = 1;
  const size_t wbytes = (size_t)c.k * ((c.Cout + 15) / 16) * (c.Cin / 64) * 1024;
  std::vector<int8_t> x((size_t)c.B * p.xbs), w(wbytes + 16), y((size_t)c.B * p.ybs);
  std::vector<std::vector<int8_t>> res(c.res, std::vector<int8_t>((size_t)c.B * p.ybs));
  std::vector<int32_t> bias(c.Cout, 3), m(c.Cout, 1 << 30), s(c.Cout, 40);
  p.x = x.data(); p.w = (int8_t*)(((uintptr_t)w.data() + 15) & ~(uintptr_t)15);
  p.bias = c.bias ? bias.data() : nullptr; p.m = m.data(); p.s = s.data(); p.y = y.data();
  if (c.res) p.res = res[0].data();
  p.n_res_more = c.res > 1 ? c.res - 1 : 0;
  for (int r = 1; r < c.res; ++r) p.res_more[r - 1] = res[r].data();
  auto& st = sim::S();
  st.regions = {{"x", (const unsigned char*)x.data(), x.size(), false}, {"w", (const unsigned char*)p.w, wbytes, false},
                {"bias", (const unsigned char*)bias.data(), bias.size() * 4, false}, {"m", (const unsigned char*)m.data(), m.size() * 4, false},
                {"s", (const unsigned char*)s.data(), s.size() * 4, false}, {"y", (const unsigned char*)y.data(), y.size(), true}};
  for (auto& r : res) st.regions.push_back({"res", (const unsigned char*)r.data(), r.size(), false});
  std::vector<uint8_t> written(y.size(), 0);
  st.written = &written;
  st.y_base = (const unsigned char*)y.data();
  std::vector<int32_t> part;
  std::vector<unsigned> count(kConvSplitCounters, 0);
  g_name = c.name;
  g_workgroups = 0;
  hipError_t e;
  auto check_output = [&](int times) {
    st.where = c.name;
    st.lane = st.wave = -1;
    size_t bytes = 0;
    for (int b = 0; b < c.B; ++b)
      for (int co = 0; co < c.Cout; ++co)
        for (int q = 0; q < p.Tout + p.ypad; ++q) {
          const int n = written[(size_t)b * p.ybs + (size_t)co * (p.Tout + p.ypad) + q];
          if (q < p.Tout ? n != times : n > times) sim::fail("item " + std::to_string(b) + " channel " + std::to_string(co) + " frame " +
                                                             std::to_string(q) + " is written " + std::to_string(n) + " times");
          bytes += q < p.Tout;
        }
    return bytes;
  };
#ifdef SIM_FEW
  {
    FewTile tile, next_tile;
    double cycles;
    if (!conv_few_cycles(p, tile, cycles) || tile.MT != t.cf_mt || tile.WC != t.cf_wc || tile.NT != t.cf_nt) sim::fail("another tile");
    t = Tuning();
    // once with the weights of a wider layer of more taps (or fewer, if those fit no tile) after it, which has tiles of its own
    // and whose lines are asked for, ...
    ConvParams next = p;
    next.Cout = 3 * c.Cout - 16; next.k = c.k + 2; next.pl = p.pl + p.dil;
    if (!conv_few_cycles(next, next_tile, cycles)) {
      next.k = c.k - 2; next.pl = p.pl - p.dil;
      if (!conv_few_cycles(next, next_tile, cycles)) sim::fail("the next layer has no tile");
    }
    const size_t nbytes = (size_t)next.k * ((next.Cout + 15) / 16) * (c.Cin / 64) * 1024;
    std::vector<int8_t> nw(nbytes + 128);
    next.w = (int8_t*)(((uintptr_t)nw.data() + 127) & ~(uintptr_t)127);
    st.regions.push_back({"next w", (const unsigned char*)next.w, nbytes, false});
    g_tuning_asked = 0;
    st.asked.clear();
    e = launch_conv_few(p, tile, &next, next_tile, nullptr);
    st.regions.pop_back();
    if (e != hipSuccess) sim::fail("the launcher does not take this case");
    check_output(1);
    check_lines(p, tile, next, next_tile, nbytes);
    std::fill(written.begin(), written.end(), 0);
    // ... and once by itself
    e = launch_conv_few(p, tile, nullptr, FewTile{}, nullptr);
    if (g_tuning_asked) sim::fail("a launch chooses a tile again");
  }
#else
  {
    if (c.s > 1) {
      p.part_bytes = 64 << 20;
      part.resize((size_t)p.part_bytes / 4);
      p.part = part.data(); p.part_count = count.data();
      st.regions.push_back({"part", (const unsigned char*)part.data(), part.size() * 4, true});
      // once as workgroups that are not the last of their tile, which store nothing of the output, ...
      g_arrival = 0;
      e = launch_conv_pipe(p, nullptr);
      for (uint8_t v : written)
        if (e != hipSuccess || v) sim::fail("a workgroup that is not the last finishes the tile");
      // ... and once as the last: every split finishes it
      g_arrival = (unsigned)c.s - 1;
    }
    e = launch_conv_pipe(p, nullptr);
  }
#endif
  if (e != hipSuccess) sim::fail("the launcher does not take this case");
  const size_t bytes = check_output(c.few || c.s < 1 ? 1 : c.s);
  std::printf("ok %-52s %ld workgroups, %zu output bytes\n", c.name, g_workgroups, bytes);
}

}  // namespace

int main() {
  const Case cases[] = {
#ifdef SIM_FEW
      //  name                                  few  a   b kg  s   B  Cin Cout   T   k st dil pl pr res bias pad
      {"few 1x1, 2 steps for 16 groups", 1, 1, 1, 0, 0, 1, 64, 64, 16, 2, 1, 1, 0, 1, 0, 1, 0},
      {"few 2x2, odd everything, dilation", 1, 2, 2, 0, 0, 2, 320, 80, 37, 17, 1, 2, 16, 16, 1, 0, 0},
      {"few 1x1 of one column, several tiles per die", 1, 1, 1, 1, 0, 2, 64, 64, 100, 3, 1, 1, 1, 1, 0, 1, 0},
#ifndef SIM_SMALL
      {"few 4x1, ring of six, three residuals", 1, 4, 1, 0, 0, 1, 320, 64, 70, 11, 1, 1, 5, 5, 3, 1, 1},
      {"few 3x2, stride 2", 1, 3, 2, 0, 0, 2, 128, 130, 99, 13, 2, 1, 6, 6, 0, 1, 0},
      {"few 1x2, long taps", 1, 1, 2, 0, 0, 1, 768, 64, 30, 77, 1, 1, 38, 38, 0, 1, 0},
      {"few 1x1, 1024 units: all of LDS", 1, 1, 1, 1, 0, 1, 1024, 64, 20, 15, 1, 7, 49, 49, 0, 1, 0},
      {"few 1x1, 60 units", 1, 1, 1, 1, 0, 2, 64, 64, 25, 14, 1, 7, 45, 46, 0, 1, 0},
      {"few 4x2, 4 frames", 1, 4, 2, 0, 0, 3, 64, 64, 4, 3, 1, 1, 1, 1, 1, 1, 1},
      {"few 1x1, 5 frames, one chunk", 1, 1, 1, 0, 0, 1, 64, 64, 5, 3, 1, 1, 1, 1, 0, 1, 0},
      {"few 1x1, 7 frames, two chunks", 1, 1, 1, 0, 0, 2, 128, 64, 7, 4, 1, 1, 2, 1, 0, 1, 0},
      {"few 2x1, 9 frames, wide padding", 1, 2, 1, 0, 0, 2, 64, 64, 9, 27, 1, 1, 13, 13, 0, 1, 0},
      {"few 2x1 of one column, rings of twelve", 1, 2, 1, 1, 0, 2, 192, 80, 41, 15, 1, 1, 7, 7, 1, 1, 0},
      {"few 4x1 of three, sums in two parts", 1, 4, 1, 3, 0, 1, 256, 112, 70, 13, 1, 1, 6, 6, 2, 1, 1},
      {"few 1x1 of three, whole rounds", 1, 1, 1, 3, 0, 1, 256, 64, 20, 16, 1, 1, 8, 7, 0, 1, 0},
      {"few 3x1, long stream", 1, 3, 1, 0, 0, 1, 512, 64, 48, 25, 1, 1, 12, 12, 0, 1, 0},
#endif
#else
      //  name                                  few  a   b kg  s   B  Cin Cout   T   k st dil pl pr res bias pad
      {"pipe 4x2, one chunk", 0, 4, 2, 1, 1, 1, 64, 96, 50, 2, 1, 1, 0, 1, 0, 1, 0},
      {"pipe 5x4, four chunks, residual", 0, 5, 4, 1, 1, 2, 256, 200, 90, 5, 1, 1, 2, 2, 1, 1, 0},
      {"pipe 4x2 two groups, odd taps", 0, 4, 2, 2, 1, 1, 320, 128, 77, 5, 1, 2, 4, 4, 0, 1, 0},
      {"pipe 4x2 four groups, one tap each, split", 0, 4, 2, 4, 3, 1, 448, 70, 60, 4, 1, 1, 1, 2, 2, 0, 1},
#ifndef SIM_SMALL
      {"pipe 10x2, two taps", 0, 10, 2, 1, 1, 1, 192, 128, 170, 2, 1, 1, 1, 0, 0, 0, 0},
      {"pipe 9x2, five chunks, 12 residuals", 0, 9, 2, 1, 1, 1, 320, 64, 150, 3, 1, 1, 1, 1, 12, 1, 1},
      {"pipe 8x4, k 3", 0, 8, 4, 1, 1, 1, 128, 256, 150, 3, 1, 1, 1, 1, 0, 1, 0},
      {"pipe 6x4, stride 2", 0, 6, 4, 1, 1, 1, 128, 256, 200, 3, 2, 1, 1, 1, 0, 1, 0},
      {"pipe 7x4, split in two", 0, 7, 4, 1, 2, 1, 192, 256, 120, 11, 1, 1, 5, 5, 1, 1, 0},
      {"pipe 6x2, split as often as chunks", 0, 6, 2, 1, 4, 2, 256, 64, 100, 3, 1, 1, 1, 1, 0, 1, 1},
      {"pipe 10x2 two groups, residual", 0, 10, 2, 2, 1, 1, 192, 128, 163, 3, 1, 1, 1, 1, 1, 1, 0},
      {"pipe 6x4 two groups, k 13", 0, 6, 4, 2, 1, 1, 384, 256, 96, 13, 1, 1, 6, 6, 0, 1, 0},
      {"pipe 8x2 two groups, fewer chunks than groups", 0, 8, 2, 2, 1, 1, 64, 128, 128, 7, 1, 1, 3, 3, 0, 0, 0},
      {"pipe 4x2 four groups, nine chunks", 0, 4, 2, 4, 1, 1, 576, 128, 64, 11, 1, 1, 5, 5, 0, 1, 0},
      {"pipe 4x4, long taps", 0, 4, 4, 1, 1, 1, 128, 256, 64, 25, 1, 3, 36, 36, 0, 1, 0},
#endif
#endif
  };
  for (const Case& c : cases) run_case(c);
  std::printf("all cases passed\n");
  return 0;
}
