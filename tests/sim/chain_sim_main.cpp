// CPU replay of the request and LDS bookkeeping of chains of pointwise layers (csrc/pw_chain.hip), in the manner of
// conv_sim_main.cpp: kernel, planner and launcher are compiled for the host against pw_pipe_sim_shim.hpp, a launch runs every
// lane of every workgroup, the lanes' records are merged per wave and replayed under in-order completion with the latest
// completion the waits allow.  Checked:
//   * every global address lies inside its operand, every LDS address inside the launch's dynamic LDS;
//   * the lanes of a wave agree on wait counts, barriers, uniform values and stores;
//   * every register that a request fills is complete when it is tied, and every one is tied; no load is outstanding when a
//     wave ends;
//   * what a wave reads of its own requests into LDS has arrived;
//   * no 16 bytes of LDS are written by one wave, by a store or by a request from its issue to the wait that completes it, and read
//     or written by another between the same two barriers;
//   * every output byte is written exactly once (pad bytes between rows at most once).
#include "pw_pipe_sim_shim.hpp"

#include <atomic>
#include <functional>
#include <map>
#include <set>
#include <type_traits>

#include "launch_shape.hpp"

// ---- host side of a launch
typedef int hipError_t;
typedef void* hipStream_t;
constexpr int hipSuccess = 0, hipErrorInvalidValue = 1;
struct dim3 {
  unsigned x, y, z;
  dim3(unsigned a, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
#define __host__
#define __builtin_amdgcn_s_barrier() sim::rec(sim::BARRIER)
#define __builtin_amdgcn_s_setprio(x) ((void)0)
#define __builtin_amdgcn_mfma_i32_4x4x4i8(a, b, c, x, y, z) (c)
#define __builtin_amdgcn_ds_bpermute(at, v) sim_bpermute(at, v)

namespace qasr {

struct Tuning {
  bool no_pw_chain = false, pw_chain_force = true;
  int chain_mt = 0;
};
inline Tuning& the_tuning() { static Tuning t; return t; }
inline const Tuning& tuning() { return the_tuning(); }

// what the layers' constants are (the same for all channels: another lane's value is known)
inline int32_t g_m = 1 << 30, g_s = 40;
inline int32_t sim_bpermute(int at, int32_t) { return at / 4 < 32 ? g_m : g_s; }

inline int32_t clamp_i8(int32_t v, int32_t lo) { return std::min(127, std::max(lo, v)); }
inline int compute_units() { return 256; }
// rows of any length: loads that the compiler waits for, stores
inline v4i load_row16(const int8_t* row, int t, int T) { sim::region_of(row + t, (size_t)std::min(16, T - t), false); return (v4i){0, 0, 0, 0}; }
inline void store_row16(int8_t* row, int t, int T, v4i) {
  if (t < T) sim::count_store(row + t, (size_t)std::min(16, T - t));
}
// LDS by ordinary accesses
inline int32_t sim_lds_const(const void* p) { sim::rec(sim::USE_LDS, (int64_t)sim::lds_off(p, 4)); return g_s; }
inline uint32_t sim_lds_word(const void* p) { sim::rec(sim::USE_LDS, (int64_t)sim::lds_off(p, 4)); return 0; }
inline void sim_lds_write4(void* p, uint32_t) { sim::rec(sim::LDS_WRITE, (int64_t)sim::lds_off(p, 4)); }
inline int32_t sim_table_code(const uint16_t* at) { sim::rec(sim::USE_LDS, (int64_t)sim::lds_off(at, 2)); return 0; }

namespace sep {
inline v2i read_tr8(const unsigned char* p) { sim::rec(sim::USE_LDS, (int64_t)sim::lds_off(p, 8)); return (v2i){0, 0}; }
inline uint32_t through_table(const unsigned char* lut, uint32_t pk) {
  for (int i = 0; i < 256; i += 16) sim::rec(sim::USE_LDS, (int64_t)sim::lds_off(lut + i, 16));
  return pk;
}
}  // namespace sep

inline hipError_t ensure_max_dynamic_lds(const void*, std::atomic<uint64_t>&) { return hipSuccess; }
void run_launch(const std::function<void()>& lane, unsigned grid, unsigned threads, size_t lds);
template <typename P>
hipError_t launch_kernel(void (*kernel)(P), dim3 grid, dim3 block, size_t shmem, hipStream_t, P p) {
  run_launch([=] { kernel(p); }, grid.x, block.x, shmem);
  return hipSuccess;
}
inline bool pw_wide_us(const ConvParams&, double&) { return false; }

}  // namespace qasr

#include "divide_extract.hpp"
#include "sep_extract.hpp"
#include "pw_chain_stripped.hpp"

namespace {

using namespace qasr;

long g_workgroups = 0;
std::string g_name;

// 16-byte blocks of LDS by barrier interval: the waves that write and read them (a wave's own order is its program's)
struct Blocks {
  std::map<std::pair<int, int64_t>, std::pair<uint32_t, uint32_t>> at;
  void touch(int wave, int from, int to, int64_t byte, int64_t bytes, bool write) {
    for (int64_t b = byte / 16; b <= (byte + bytes - 1) / 16; ++b)
      for (int i = from; i <= to; ++i) (write ? at[{i, b}].first : at[{i, b}].second) |= 1u << wave;
  }
  void check() const {
    for (const auto& [key, use] : at) {
      const uint32_t w = use.first, all = w | use.second;
      if (w && (all & (all - 1))) sim::fail("LDS block " + std::to_string(key.second) + " is shared between waves without a barrier");
    }
  }
};

struct Req { sim::Kind k; int64_t a, b; int interval; bool done; };

void replay(int wave, const std::vector<sim::Ev>& ev, const std::vector<std::vector<sim::Ev>>& lanes, Blocks& blocks) {
  std::vector<Req> reqs;
  size_t head = 0;
  std::map<int64_t, size_t> reg_req;
  std::set<int64_t> tied;
  std::map<int64_t, size_t> lands;                  // 16-byte block of LDS -> the youngest request that fills it
  int interval = 0;
  for (size_t n = 0; n < ev.size(); ++n) {
    const sim::Ev& e = ev[n];
    switch (e.k) {
      case sim::ISSUE_LDS:
        for (int64_t b = e.a / 16; b <= (e.a + e.b - 1) / 16; ++b) lands[b] = reqs.size();
        reqs.push_back(Req{e.k, e.a, e.b, interval, false});
        break;
      case sim::ISSUE_REG: reg_req[e.a] = reqs.size(); reqs.push_back(Req{e.k, 0, 0, interval, false}); break;
      case sim::STORE: reqs.push_back(Req{e.k, 0, 0, interval, false}); break;
      case sim::WAIT:
        while (reqs.size() - head > (size_t)e.a) {
          Req& r = reqs[head++];
          r.done = true;
          if (r.k == sim::ISSUE_LDS) blocks.touch(wave, r.interval, interval, r.a, r.b, true);
        }
        break;
      case sim::USE_REG: {
        auto it = reg_req.find(e.a);
        if (it == reg_req.end()) sim::fail("tie of a register no load was issued for");
        if (!reqs[it->second].done) sim::fail("a register is used before its load has completed");
        tied.insert(e.a);
        break;
      }
      case sim::USE_LDS:
      case sim::LDS_WRITE:
        for (const sim::Ev& l : lanes[n]) {
          blocks.touch(wave, interval, interval, l.a, 1, e.k == sim::LDS_WRITE);
          const auto it = lands.find(l.a / 16);
          if (it != lands.end() && !reqs[it->second].done) sim::fail("LDS is read or written where a request of the wave has not arrived");
        }
        break;
      case sim::BARRIER: ++interval; break;
      default: break;
    }
  }
  for (size_t i = head; i < reqs.size(); ++i)
    if (reqs[i].k != sim::STORE) sim::fail("loads are outstanding when the wave ends");
  if (tied.size() != reg_req.size()) sim::fail("a register that a load fills is never tied");
}

}  // namespace

void qasr::run_launch(const std::function<void()>& lane, unsigned grid, unsigned threads, size_t lds_size) {
  auto& st = sim::S();
  for (unsigned wg = 0; wg < grid; ++wg) {
    std::vector<unsigned char> lds(lds_size, 0);
    st.lds = lds.data(); st.lds_bytes = lds_size;
    blockIdx.x = wg;
    st.where = g_name + " workgroup " + std::to_string(wg);
    Blocks blocks;
    bool any = false;
    for (unsigned wv = 0; wv < threads / 64; ++wv) {
      sim::Wave w;
      w.lanes.resize(64);
      for (int l = 0; l < 64; ++l) {
        st.ev.clear(); st.dwords.clear(); st.lane = l; st.wave = (int)wv; st.next_uid = 1;
        threadIdx.x = wv * 64 + (unsigned)l;
        lane();
        w.lanes[l] = st.ev;
      }
      st.lane = -1;
      std::vector<std::vector<sim::Ev>> lanes;
      const std::vector<sim::Ev> ev = sim::merge(w, &lanes);
      replay((int)wv, ev, lanes, blocks);
      any = any || ev.size() > 1;
    }
    blocks.check();
    g_workgroups += any;
  }
}

namespace {

struct Case {
  const char* name;
  int MT, B, T, dw;                  // dw: taps of the depthwise layer in front, 0 without one
  std::vector<int> widths;
  int bias, act, glu, in_pad, out_pad, s;   // act: table after every layer but the last (and after the depthwise one)
};

struct Layer { std::vector<int8_t> w; std::vector<int32_t> bias, m, s; std::vector<uint8_t> table; };

void run_case(const Case& c) {
  the_tuning() = Tuning();
  the_tuning().chain_mt = c.MT;
  g_s = c.s;
  const int n = (int)c.widths.size() - 1, pitch = (c.T + 15) / 16 * 16;
  const int xpitch = c.in_pad ? pitch : c.T, ypitch = c.out_pad ? pitch : c.T;
  const int in_ch = c.widths[0], out_ch = c.glu ? c.widths[n] / 2 : c.widths[n];
  const int64_t xbs = (int64_t)in_ch * xpitch, ybs = (int64_t)c.widths[n] * ypitch;
  std::vector<int8_t> x((size_t)(c.B * xbs) + 16), y((size_t)(c.B * ybs) + 16);
  auto aligned = [](std::vector<int8_t>& v) { return (int8_t*)(((uintptr_t)v.data() + 15) & ~(uintptr_t)15); };
  int8_t *const xa = aligned(x), *const ya = aligned(y);
  auto& st = sim::S();
  st.regions = {{"x", (const unsigned char*)xa, (size_t)(c.B * xbs), false}, {"y", (const unsigned char*)ya, (size_t)(c.B * ybs), true}};
  std::vector<Layer> layers(n + 1);                 // (the depthwise one last)
  ChainOp op[kMaxChain]{};
  auto fill = [&](Layer& l, size_t wbytes, int cout, bool table) {
    l.w.assign(wbytes + 16, 1);
    l.bias.assign(cout + 4, 3); l.m.assign(cout + 4, g_m); l.s.assign(cout + 4, c.s); l.table.assign(512, 1);
    auto ints = [](std::vector<int32_t>& v) { return (int32_t*)(((uintptr_t)v.data() + 15) & ~(uintptr_t)15); };
    st.regions.push_back({"w", (const unsigned char*)aligned(l.w), wbytes, false});
    for (auto* v : {&l.bias, &l.m, &l.s}) st.regions.push_back({"constants", (const unsigned char*)ints(*v), (size_t)cout * 4, false});
    if (table) st.regions.push_back({"table", l.table.data(), l.table.size(), false});
    ConvParams p{};
    p.w = aligned(l.w); p.bias = c.bias ? ints(l.bias) : nullptr; p.m = ints(l.m); p.s = ints(l.s);
    p.B = c.B; p.k = 1; p.stride = p.dil = 1; p.w_packed = 1;
    return p;
  };
  for (int i = 0; i < n; ++i) {
    const int cin = c.widths[i], cout = c.widths[i + 1];
    const bool glu = c.glu && i + 1 == n, act = c.act && i + 1 < n;
    ConvParams& p = op[i].p = fill(layers[i], (size_t)cin * cout, cout, glu || act);
    p.Cin = cin; p.Cout = cout; p.relu = i & 1;
    // (as an encoder has them: rows of the slots' pitch inside, and over the pitch where a layer's input and output have one)
    const int in = i || c.dw ? pitch : xpitch, out = i + 1 < n ? pitch : ypitch;
    p.Tin = p.Tout = in == out ? in : c.T;
    p.xpad = in - p.Tin; p.ypad = out - p.Tout;
    p.xbs = (int64_t)cin * in; p.ybs = (int64_t)cout * out;
    op[i].glu = glu;
    op[i].table = glu || act ? layers[i].table.data() : nullptr;
    op[i].glu_m = glu ? 1 << 30 : 0; op[i].glu_s = glu ? (c.glu == 2 ? 30 : 45) : 1;
  }
  op[0].p.x = xa;
  op[n - 1].p.y = ya;
  ConvParams d{};
  std::vector<uint32_t> img(512 * 3 * 4 + 4);
  const uint32_t* const image = (const uint32_t*)(((uintptr_t)img.data() + 15) & ~(uintptr_t)15);
  if (c.dw) {
    d = fill(layers[n], (size_t)512 * c.dw, 512, c.act);
    st.regions.push_back({"image", (const unsigned char*)image, (size_t)512 * 3 * 16, false});
    d.depthwise = 1; d.Cin = d.Cout = 512; d.Tin = d.Tout = c.T; d.k = c.dw; d.pl = (c.dw - 1) / 2; d.w_packed = 0; d.relu = c.dw & 1;
    d.xpad = xpitch - c.T; d.ypad = pitch - c.T;
    d.xbs = xbs; d.ybs = (int64_t)512 * pitch;
    d.x = xa;
    d.act_lut = c.act ? layers[n].table.data() : nullptr;
    op[0].p.x = nullptr;
  }
  std::vector<uint8_t> written((size_t)(c.B * ybs), 0);
  st.written = &written;
  st.y_base = (const unsigned char*)ya;
  g_name = c.name;
  g_workgroups = 0;
  const hipError_t e = launch_pw_chain(c.dw ? &d : nullptr, image, op, n, nullptr);
  st.where = c.name;
  st.lane = st.wave = -1;
  if (e != hipSuccess) sim::fail("the launcher does not take this case");
  size_t bytes = 0;
  for (int b = 0; b < c.B; ++b)
    for (int co = 0; co < c.widths[n]; ++co)
      for (int q = 0; q < ypitch; ++q) {
        const int k = written[(size_t)(b * ybs) + (size_t)co * ypitch + q];
        const bool out = q < c.T && co < out_ch;
        if (out ? k != 1 : co < out_ch ? k > 1 : k != 0)
          sim::fail("item " + std::to_string(b) + " channel " + std::to_string(co) + " frame " + std::to_string(q) + " is written " +
                    std::to_string(k) + " times");
        bytes += out;
      }
  std::printf("ok %-56s %ld workgroups, %zu output bytes\n", c.name, g_workgroups, bytes);
}

}  // namespace

int main() {
  const Case cases[] = {
      //  name                                       MT  B   T  dw  widths                    bias act glu in out  s
      {"two layers, whole rows", 1, 1, 32, 0, {512, 512, 512}, 1, 0, 0, 1, 1, 40},
      {"three layers, two groups, odd rows", 2, 1, 45, 0, {1024, 512, 1536, 512}, 0, 0, 0, 0, 0, 40},
      {"depthwise layer, two passes, GLU", 2, 2, 33, 32, {512, 512, 1024}, 1, 1, 1, 1, 1, 40},
#ifndef SIM_SMALL
      {"four layers with activations, 64-bit rescale", 1, 1, 17, 0, {512, 1024, 512, 512, 512}, 1, 1, 0, 0, 1, 20},
      {"two groups, one left over in every item", 2, 3, 80, 0, {512, 512, 512}, 1, 0, 0, 1, 0, 62},
      {"wide layers", 1, 1, 16, 0, {2048, 512, 2048}, 1, 0, 0, 1, 1, 40},
      {"depthwise layer, one group, long taps", 1, 1, 50, 42, {512, 512, 512}, 0, 0, 0, 1, 0, 40},
      {"depthwise layer, a Conformer's, short rescale of GLU", 1, 2, 20, 31, {512, 512, 2048, 512, 1024}, 1, 1, 2, 1, 1, 40},
      {"depthwise layer, three taps, 64-bit rescale", 2, 1, 31, 3, {512, 512, 1024}, 1, 0, 0, 1, 0, 20},
      {"more tiles than dies", 2, 9, 48, 0, {512, 512, 512}, 0, 1, 1, 1, 1, 40},
#endif
  };
  for (const Case& c : cases) run_case(c);
  std::printf("all cases passed\n");
  return 0;
}
