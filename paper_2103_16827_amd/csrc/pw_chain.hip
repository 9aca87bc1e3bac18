// Consecutive pointwise (k = 1) layers in one launch, with a depthwise layer in front of them where there is one: from a
// Conformer's depthwise convolution over the next layer's two feed-forward products to its first pointwise layer.
//
// Frames are independent here, so a workgroup of 16 waves can take its one or two 16-frame groups through all layers: the
// tensors between them, up to 2048 channels wide, stay in LDS, four launches and the chains of first loads in front of each of
// them (about 5 us) become one.  What bounds it is the weights: every workgroup streams all of them once, 64 bytes per
// cycle of its unit's path from the L2 (2.75 MiB, by the counters 3.2 MB with rows and constants: 21 us of the 32 to 36 it takes,
// 91 % of them out of the L2; the products, which pass under it, are 8 us of the matrix pipes), so it pays while the frames make
// few tiles for each unit.  Therefore
//   - a wave's weights are ONE stream over layers, passes and blocks, requested 8 steps ahead by hand (vmem.hpp) across
//     every epilogue and barrier; barriers stand between layers only, and wait for LDS alone;
//   - workgroups take passes and blocks in different orders (turned below): in step, all of a die's would miss its L2 on the same
//     lines at the same time (34.7 -> 32.3 us with 16 frames per workgroup, 38.0 -> 37.0 with 32);
//   - a wave behind the others goes first at the address path, which serves the oldest wave otherwise: they drifted 10 k cycles
//     apart over four passes, and the stream ran dry at the layer's end (32.3 -> 31.6, 37.0 -> 35.7 us).
// Per layer of the Conformer-L-shaped network, us, launch by launch / as chains (4 layers, 17 to 20 launches / 5): 16 x 400
// frames 42.3 / 35.4, with Swish and GLU 48.6 / 36.2; 8 x 400 36.1 / 33.0 and 40.6 / 33.0.  Four 512 -> 512 layers, 16 x 400: 28.5 / 16.9.
// Tried: a barrier per block (slower, 36.1 against 33.7), weights brought into the L2 ahead of use by a dword per line (no gain).
//
// LDS: the input of layer l in one of two buffers by its parity, a plane [channel][16 frames] for each group: transposing reads and
// the dwords of finished blocks both touch contiguous bytes.  A layer's products read one buffer, its finished blocks go to the other.
#include "pw_chain.hpp"
#include "kernels.hpp"
#include "launch_shape.hpp"
#include "sep_body.hpp"
#include "tuning.hpp"
#include "vmem.hpp"

namespace qasr {

namespace {

using sep::v4u;
using sep::DwSmall;
using sep::read_tr8;
using sep::through_table;
using sep::kStoreThrough;

constexpr int kWaves = 16;
constexpr int D = 8;                 // steps (of 64 input channels) per block = weights on their way

// value bytes times the sigmoid codes of the gate bytes, rescaled
template <bool HIGH>
__device__ __forceinline__ uint32_t glu4(uint32_t a, uint32_t g, const uint16_t* table, int32_t m, int32_t s) {
  const uint32_t gc = g ^ 0x80808080u;
  uint32_t pk = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int32_t v = (int32_t)(int8_t)(a >> (8 * e)) * (int32_t)table[(gc >> (8 * e)) & 0xffu];
    const int32_t r = HIGH ? ((int32_t)__mulhi(v, m) + (1 << ((s - 33) & 31))) >> ((s - 32) & 31) : dyadic_rescale64(v, m, s);
    pk |= ((uint32_t)clamp_i8(r, -128) & 0xffu) << (8 * e);
  }
  return pk;
}

// requests of the weights of step I (of a block of D) of two columns
template <int I>
__device__ __forceinline__ void load_step(v4i (&r)[2], const int8_t* w0, const int8_t* w1, uint32_t wlane) {
  gload16_into<(I & 3) * 1024>(r[0], w0 + (I >> 2) * 4096, wlane);
  gload16_into<(I & 3) * 1024>(r[1], w1 + (I >> 2) * 4096, wlane);
}
template <int I, int N>
__device__ __forceinline__ void load_steps(v4i (&wb)[D][2], const int8_t* w0, const int8_t* w1, uint32_t wlane) {
  if constexpr (I < N) {
    load_step<I>(wb[I], w0, w1, wlane);
    load_steps<I + 1, N>(wb, w0, w1, wlane);
  }
}

constexpr int AH = 2, AR = AH + 1;   // activation operands read ahead

// Items I .. of a block: item = unit I % MT of step I / MT.  MORE: the next block's weights are requested as the steps' registers
// become free.
template <int MT, bool MORE, int I>
__device__ __forceinline__ void items(v4i (&acc)[MT][2], v4i (&wb)[D][2], v2i (&ar)[AR][2], const unsigned char* a0, int plane,
                                      const int8_t* w0, const int8_t* w1, uint32_t wlane) {
  if constexpr (I < D * MT) {
    constexpr int st = I / MT, mt = I % MT;
    if constexpr (mt == 0) {
      wait_vm<MORE ? 2 * (D - 1) : 2 * (D - 1 - st)>();
      tie(wb[st][0]);
      tie(wb[st][1]);
    }
    const v4i a = {ar[I % AR][0].x, ar[I % AR][0].y, ar[I % AR][1].x, ar[I % AR][1].y};
    if constexpr (I + AH < D * MT) {
      const unsigned char* const r = a0 + ((I + AH) % MT) * plane + ((I + AH) / MT) * 1024;
      ar[(I + AH) % AR][0] = read_tr8(r);
      ar[(I + AH) % AR][1] = read_tr8(r + 512);
    }
    acc[mt][0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, wb[st][0], acc[mt][0], 0, 0, 0);
    acc[mt][1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, wb[st][1], acc[mt][1], 0, 0, 0);
    if constexpr (MORE && mt == MT - 1) load_step<st>(wb[st], w0, w1, wlane);
    __builtin_amdgcn_sched_barrier(0);
    items<MT, MORE, I + 1>(acc, wb, ar, a0, plane, w0, w1, wlane);
  }
}

// NA: quads of taps of the depthwise layer in front, 0 without one
template <int MT, int NA>
__global__ __launch_bounds__(64 * kWaves) void pw_chain_kernel(ChainParams p) {
  extern __shared__ __align__(128) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // (every line of the arguments is asked for in one go)
  asm volatile("" ::"s"(p.dw.x), "s"(p.dw.xbs), "s"(p.dw.xpitch), "s"(p.dw.Tin), "s"(p.y), "s"(p.ybs), "s"(p.n), "s"(p.tpr), "s"(p.g_base), "s"(p.g_more),
               "s"(p.wgs), "s"(p.per_xcd), "s"(p.const_off), "s"(p.rows_off), "s"(p.r_tpr));
  if constexpr (NA > 0)
    asm volatile("" ::"s"(p.dw.img), "s"(p.dw.dbias), "s"(p.dw.dm), "s"(p.dw.ds), "s"(p.dw.lut), "s"(p.dw.o16), "s"(p.dw.units), "s"(p.dw.units_inv));
#pragma unroll
  for (int l = 0; l < kMaxChain; ++l) asm volatile("" ::"s"(p.layer[l].w), "s"(p.layer[l].cin));
  const int v = (int)(blockIdx.x & 7) * p.per_xcd + (int)(blockIdx.x >> 3);
  if (v >= p.wgs || (int)(blockIdx.x >> 3) >= p.per_xcd) return;             // whole workgroup
  const int b = divide_uniform24(v, p.tpr, p.r_tpr), ti = v - b * p.tpr;
  const int g0 = ti * p.g_base + min(ti, p.g_more), gn = p.g_base + (ti < p.g_more ? 1 : 0);   // <= MT

  // ---- what the first layer reads: a plane of 16 bytes per row for each unit
  constexpr int CPW = 512 / kWaves;                 // depthwise channels of a wave
  using Dw = DwSmall<CPW, MT, NA ? NA : 3, false>;
  Dw dw;
  uint32_t in = 0, last = 0;                        // bit j: chunk j has frames; ... and its row ends inside it
  unsigned char* const rows = lds + p.rows_off + wave * p.row_bytes;
  unsigned char* const lut = rows + p.row_bytes - 256;
  unsigned char* const taps = lds + p.taps_off + wave * (CPW * (NA ? NA : 3) * 16);
  if constexpr (NA > 0) {
    // as DwSmall::load and lay, but straight into LDS; what lies outside the rows is put right after the wait
    const int8_t* const xw = p.dw.x + (int64_t)b * p.dw.xbs + (int64_t)(wave * CPW) * p.dw.xpitch;
#pragma unroll
    for (int j = 0; j < Dw::NL; ++j) {
      const int L = lane + 64 * j, ch = (L * p.dw.units_inv) >> 16, t = 16 * (g0 + p.dw.o16 + L - ch * p.dw.units);
      const bool on = t >= 0 && t < p.dw.Tin;
      if (on) in |= 1u << j;
      if (t == (p.dw.Tin & ~15)) last |= 1u << j;
      if (L < CPW * p.dw.units) direct_load16(xw + (on ? ch * p.dw.xpitch + t : 0), rows + 1024 * j);
    }
#pragma unroll
    for (int j = 0; j < Dw::NWL; ++j)
      if (lane + 64 * j < CPW * NA) direct_load16(reinterpret_cast<const v4i*>(p.dw.img) + wave * CPW * NA + lane + 64 * j, taps + 1024 * j);
    dw.dc.load_by_hand(p.dw.dm, p.dw.ds, p.dw.dbias, wave * CPW, lane);
    if (p.dw.lut) direct_load4(p.dw.lut + 4 * lane, lut);
  } else {
    const int8_t* const xb = p.dw.x + (int64_t)b * p.dw.xbs;
    const int rows0 = p.layer[0].cin;
    if (p.xragged) {
      const int u = tid % MT, t = 16 * (g0 + u);
      if (u < gn)
        for (int r = tid / MT; r < rows0; r += 1024 / MT)
          *reinterpret_cast<v4i*>(lds + p.buf[0] + u * (rows0 * 16) + r * 16) = load_row16(xb + (int64_t)r * p.dw.xpitch, t, p.dw.Tin);
    } else {
      for (int j = wave; j < rows0 / 64 * gn; j += kWaves) {    // (uniform) 64 rows of a unit at a time
        const int u = gn == 1 ? 0 : j & 1, r = (gn == 1 ? j : j >> 1) * 64;
        direct_load16(xb + (int64_t)(r + lane) * p.dw.xpitch + 16 * (g0 + u), lds + p.buf[0] + u * (rows0 * 16) + r * 16);
      }
    }
  }
  // ---- the wave's weights: one stream over all layers, passes and blocks of D steps
  struct At { int l, pass, kb; };                   // a block of the stream
  const int rank = (int)(blockIdx.x >> 3);          // among the die's workgroups
  auto turned = [&](int i, int n) __attribute__((always_inline)) { return (n & (n - 1)) ? i : (i + rank) & (n - 1); };
  auto columns = [&](const ChainLayer& q, int pass, int& c0, int& c1) __attribute__((always_inline)) {
    const int ps = turned(pass, q.cout / 512);
    c0 = q.glu ? ps * kWaves + wave : 2 * (ps * kWaves + wave);
    c1 = q.glu ? c0 + q.cout / 32 : c0 + 1;
  };
  auto weights = [&](const At& a, const int8_t*& w0, const int8_t*& w1) __attribute__((always_inline)) {
    const ChainLayer& q = p.layer[a.l];
    const int kch = q.cin / 64, kb = turned(a.kb, q.cin / 512);
    int c0, c1;
    columns(q, a.pass, c0, c1);
    w0 = q.w + ((int64_t)c0 * kch + kb * D) * 1024;
    w1 = q.w + ((int64_t)c1 * kch + kb * D) * 1024;
  };
  auto next = [&](At& a) __attribute__((always_inline)) {
    const ChainLayer& q = p.layer[a.l];
    if (++a.kb * (D * 64) < q.cin) return;
    a.kb = 0;
    if (++a.pass * 512 < q.cout) return;
    a.pass = 0;
    ++a.l;
  };
  const uint32_t wlane = (uint32_t)lane * 16;
  const int8_t *w0, *w1;
  At cur{0, 0, 0};
  v4i wb[D][2];
#pragma unroll
  for (int i = 0; i < D; ++i) wb[i][0] = wb[i][1] = (v4i){0, 0, 0, 0};
  weights(cur, w0, w1);
  __builtin_amdgcn_s_barrier();                     // (no wave's first loads queue behind another's weights)
  load_steps<0, D / 2>(wb, w0, w1, wlane);
  // ---- constants of layer after layer, bias | m | s, 256 channels (8 pieces at most) by a wave
  {
    unsigned char* dst = lds + p.const_off;
#pragma unroll
    for (int l = 0; l < kMaxChain; ++l) {
      if (l < p.n) {
        const ChainLayer& q = p.layer[l];
#pragma unroll
        for (int which = 0; which < 3; ++which) {
          const int c = (wave & 7) * 256;
          if (wave >> 3 == ((3 * l + which) & 1) && c < q.cout) {             // (uniform)
            const int32_t* const src = which == 0 ? q.bias : which == 1 ? q.m : q.s;
            unsigned char* const to = dst + which * 4 * q.cout + 4 * c;
            if (!src) {
              *reinterpret_cast<v4i*>(to + 16 * lane) = (v4i){0, 0, 0, 0};
            } else {
              direct_load16(src + c + 4 * lane, to);
            }
          }
        }
        if (q.table && wave == kWaves - 1 - l) {
          direct_load4(q.table + 4 * lane, lds + p.table_off + 512 * l);
          if (q.glu) direct_load4(q.table + 256 + 4 * lane, lds + p.table_off + 512 * l + 256);
        }
        dst += 12 * q.cout;
      }
    }
  }
  if constexpr (NA > 0) {
    wait_vm<D>();                                   // (and as many of the weights as other requests came after)
    tie(dw.dc.ms);
    tie(dw.dc.b);
#pragma unroll
    for (int j = 0; j < Dw::NL; ++j)
      if (lane + 64 * j < CPW * p.dw.units) {
        v4i* const c = reinterpret_cast<v4i*>(rows + 16 * (lane + 64 * j));
        if (!(in & (1u << j))) *c = (v4i){0, 0, 0, 0};
        else if (last & (1u << j)) *c = keep_bytes(*c, p.dw.Tin & 15);
      }
    asm volatile("" ::: "memory");                  // (lanes read what other lanes of the wave wrote: LDS is in order)
    // (one block of 16 channels after the other: the weights on their way hold half of the registers)
#pragma unroll
    for (int blk = 0; blk < CPW / 16; ++blk) {
      v4i dacc[1][MT];
      dw.template multiply<1>(p.dw, p.dw.units, rows, taps, lane, blk, dacc);
      unsigned char* const to = lds + p.buf[0] + (wave * CPW + (lane >> 2)) * 16 + 4 * (lane & 3);
      dw.template finish<1>(p.dw, lut, lane, blk, dacc, [&](int bk, int q, uint32_t pk) __attribute__((always_inline)) {
        *reinterpret_cast<uint32_t*>(to + q * 8192 + bk * 256) = pk;
      });
    }
  }
  load_steps<D / 2, D>(wb, w0, w1, wlane);
  wait_vm<D>();                                     // tile, constants and tables have arrived
  const int n = lane & 15, gi = lane >> 4, jr = n >> 1;
  const uint32_t arow = (uint32_t)((8 * gi + jr) * 16 + 8 * (n & 1));
  int const_off = p.const_off;
  v4i acc[MT][2];
  v2i ar[AR][2];
  const unsigned char* a0;
  auto barrier = [&]() __attribute__((always_inline)) {     // (LDS only: the weights stay on their way)
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  auto begin_pass = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt][0] = acc[mt][1] = (v4i){0, 0, 0, 0};
  };
  auto first_items = [&]() __attribute__((always_inline)) {
    const int plane = p.layer[cur.l].cin * 16;
    a0 = lds + p.buf[cur.l & 1] + turned(cur.kb, p.layer[cur.l].cin / 512) * (D * 1024) + arow;
#pragma unroll
    for (int i = 0; i < AH; ++i) {
      const unsigned char* const r = a0 + (i % MT) * plane + (i / MT) * 1024;
      ar[i][0] = read_tr8(r);
      ar[i][1] = read_tr8(r + 512);
    }
  };
  auto end_pass = [&]() __attribute__((always_inline)) {
    const ChainLayer& q = p.layer[cur.l];
    int c0, c1;
    columns(q, cur.pass, c0, c1);
    const int cout = q.cout, plane = (q.glu ? cout / 2 : cout) * 16;
    const unsigned char* const cst = lds + const_off + 4 * n;
    const int32_t b0 = *reinterpret_cast<const int32_t*>(cst + 64 * c0), b1 = *reinterpret_cast<const int32_t*>(cst + 64 * c1);
    const int32_t m0 = *reinterpret_cast<const int32_t*>(cst + 4 * cout + 64 * c0), m1 = *reinterpret_cast<const int32_t*>(cst + 4 * cout + 64 * c1);
    const int32_t s0 = *reinterpret_cast<const int32_t*>(cst + 8 * cout + 64 * c0), s1 = *reinterpret_cast<const int32_t*>(cst + 8 * cout + 64 * c1);
    const bool fast = __all(s0 >= kShortMin && s0 <= kShortMax && s1 >= kShortMin && s1 <= kShortMax);
    const unsigned char* const table = lds + p.table_off + 512 * cur.l;
    unsigned char* const out = lds + p.buf[(cur.l + 1) & 1];
    auto finish = [&](auto fast_tag, auto relu_tag) __attribute__((always_inline)) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        uint32_t pk[2];
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
          const int32_t bv = nt ? b1 : b0;
          const int32_t a4[4] = {acc[mt][nt][0] + bv, acc[mt][nt][1] + bv, acc[mt][nt][2] + bv, acc[mt][nt][3] + bv};
          const int32_t m = nt ? m1 : m0, s = nt ? s1 : s0;
          if constexpr (decltype(fast_tag)::value)
            pk[nt] = requant_short4<false, decltype(relu_tag)::value>(a4, m, s - 32, 1 << ((s - 33) & 31), 0u);
          else
            pk[nt] = requant_pack4<false, false>(a4, m, s, 0, 0u, q.relu ? 0 : -128, 127);
        }
        unsigned char* const o = out + mt * plane + 16 * n + 4 * gi;
        if (q.glu) {
          const uint16_t* const codes = reinterpret_cast<const uint16_t*>(table);
          *reinterpret_cast<uint32_t*>(o + 256 * c0) = q.glu_s >= 33 ? glu4<true>(pk[0], pk[1], codes, q.glu_m, q.glu_s)
                                                                     : glu4<false>(pk[0], pk[1], codes, q.glu_m, q.glu_s);
        } else {
          if (q.table) {
            pk[0] = through_table(table, pk[0]);
            pk[1] = through_table(table, pk[1]);
          }
          *reinterpret_cast<uint32_t*>(o + 256 * c0) = pk[0];
          *reinterpret_cast<uint32_t*>(o + 256 * c1) = pk[1];
        }
      }
    };
    if (!fast) finish(std::false_type{}, std::false_type{});
    else if (q.relu) finish(std::true_type{}, std::true_type{});
    else finish(std::true_type{}, std::false_type{});
    if (cur.l + 1 < p.n) return;
    // out: the wave's own rows, lane -> unit lane % MT of row lane / MT
    asm volatile("" ::: "memory");
    const int u = lane % MT, row = lane / MT, t = 16 * (g0 + u);
    const bool ok = row < (q.glu ? 16 : 32) && u < gn;
    const v4i o = *reinterpret_cast<const v4i*>(out + (ok ? u * plane + 256 * c0 + 16 * row : 0));
    int8_t* const yb = p.y + (int64_t)b * p.ybs;
    if (p.yragged) {
      if (ok) store_row16(yb + (int64_t)(16 * c0 + row) * p.ypitch, t, p.Tout, o);
    } else {
      const __amdgpu_buffer_rsrc_t yrs = __builtin_amdgcn_make_buffer_rsrc(yb, 0, 0x7ffffff0, 0x00027000);
      const v4u ov = {(unsigned)o.x, (unsigned)o.y, (unsigned)o.z, (unsigned)o.w};
      __builtin_amdgcn_raw_buffer_store_b128(ov, yrs, ok ? (uint32_t)(16 * c0 + row) * (uint32_t)p.ypitch + (uint32_t)t : 0xfffffff0u, 0,
                                             kStoreThrough);
    }
  };
  barrier();
  begin_pass();
  for (int left = p.blocks - 1; left > 0; --left) {
    At ahead = cur;
    next(ahead);
    weights(ahead, w0, w1);
    first_items();
    items<MT, true, 0>(acc, wb, ar, a0, p.layer[cur.l].cin * 16, w0, w1, wlane);
    const bool layer_end = ahead.kb == 0 && ahead.pass == 0;
    if (ahead.kb == 0) {
      end_pass();
      if (ahead.pass == 0) const_off += 12 * p.layer[cur.l].cout;
      begin_pass();
    }
    cur = ahead;
    if (layer_end) barrier();
    switch (cur.pass + cur.kb) {
      case 0: __builtin_amdgcn_s_setprio(3); break;
      case 1: __builtin_amdgcn_s_setprio(2); break;
      case 2: __builtin_amdgcn_s_setprio(1); break;
      default: __builtin_amdgcn_s_setprio(0);
    }
  }
  first_items();
  items<MT, false, 0>(acc, wb, ar, a0, p.layer[cur.l].cin * 16, w0, w1, wlane);
  wait_vm<0>();
  end_pass();
}

struct Plan { int MT, NA, buf[2], const_off, table_off, rows_off, row_bytes, taps_off, lds; int64_t wgs; DwParams dw; };

bool plan(const ConvParams* dw, const ChainOp* op, int n, int cus, Plan& pl) {
  if (tuning().no_pw_chain || n < 2 || n > kMaxChain) return false;
  const ConvParams &f = op[0].p, &e = op[n - 1].p;
  int consts = 0;
  for (int i = 0; i < n; ++i) {
    const ConvParams& p = op[i].p;
    if (p.depthwise || p.k != 1 || p.stride != 1 || p.pl != 0 || p.Tout != p.Tin || !p.w_packed || (uintptr_t)p.w % 16 || p.res ||
        p.n_res_more || p.B != f.B || (p.Tout + 15) / 16 != (f.Tin + 15) / 16)
      return false;
    if (p.Cin % 512 || p.Cin > 2048 || p.Cout % 512 || p.Cout > 2048) return false;
    if ((uintptr_t)p.bias % 16 || (uintptr_t)p.m % 16 || (uintptr_t)p.s % 16) return false;
    if (i > 0 && p.Cin != op[i - 1].p.Cout) return false;
    if (op[i].glu && i + 1 < n) return false;
    consts += 12 * p.Cout;
  }
  if (f.Tin < 4 || e.Tout < 4 || (int64_t)e.Cout * (e.Tout + e.ypad) > 0x7fffff00LL) return false;
  if (dw && (f.Cin != 512 || dw->Cout != f.Cin || dw->B != f.B || (dw->Tout + 15) / 16 != (f.Tin + 15) / 16)) return false;
  const int gpr = (f.Tin + 15) / 16;
  bool found = false;
  for (int MT = 1; MT <= 2; ++MT) {
    if (tuning().chain_mt && MT != tuning().chain_mt) continue;
    Plan c{};
    c.MT = MT;
    int size[2] = {0, 0};
    for (int i = 0; i <= n; ++i) {
      const int ch = i < n ? op[i].p.Cin : e.Cout;
      if (ch * 16 * MT > size[i & 1]) size[i & 1] = ch * 16 * MT;
    }
    c.buf[0] = 0;
    c.buf[1] = size[0];
    c.const_off = size[0] + size[1];
    if (dw) {                                       // its scratch lies over what is written later
      if (!dw_small_params(*dw, MT, c.dw, c.NA) || c.NA != 3) continue;
      c.rows_off = 512 * 16 * MT;
      c.row_bytes = sep::small_row_bytes(32, c.dw.units, MT, c.NA) + 256;
      c.taps_off = c.rows_off + kWaves * c.row_bytes;
      const int end = c.taps_off + 512 * 16 * c.NA;
      if (end > c.const_off) c.const_off = end;
    }
    c.table_off = c.const_off + consts;
    c.lds = c.table_off + 512 * n;
    if (c.lds > 160 * 1024) continue;
    c.wgs = (int64_t)f.B * ((gpr + MT - 1) / MT);
    if (c.wgs > max_workgroups(1024) || c.wgs >= 1 << 24) continue;
    if (found && (c.wgs + cus - 1) / cus >= (pl.wgs + cus - 1) / cus) continue;   // (the same rounds: fewer products)
    pl = c;
    found = true;
  }
  return found;
}

bool ragged(int64_t pitch, int64_t bs, const int8_t* at) { return pitch % 16 || bs % 16 || (uintptr_t)at % 16; }

template <int MT, int NA>
hipError_t launch_t(const ChainParams& p, size_t lds, hipStream_t st) {
  static std::atomic<uint64_t> lds_raised{0};       // per instantiation, a bit per device
  if (const hipError_t e = ensure_max_dynamic_lds((const void*)pw_chain_kernel<MT, NA>, lds_raised); e != hipSuccess) return e;
  return launch_kernel(pw_chain_kernel<MT, NA>, dim3((unsigned)(8 * p.per_xcd)), dim3(64 * kWaves), lds, st, p);
}

}  // namespace

bool pw_chain_supported(const ChainOp* op, int n) {
  Plan pl;
  return plan(nullptr, op, n, 256, pl);
}

// The chain's time, a fixed part and the stream (blocks of 256 KiB), against its layers' by pw_wide's model.  It takes launches
// whose workgroups run at once, one per unit: 256 tiles, which a batch item's frames begin anew (20 x 400 frames are 260 of two
// groups); a second round streams all weights again, 1.03 to 1.6 of the separate launches.  Rows of more than 512 channels are not
// written under the last pass, 1 us per 512 more (512 -> 512 -> 1024 at 4 x 800 frames 12.8 us as a chain, 12.2 apart); where a
// chain of two layers, which saves one launch only, has two groups per workgroup, 2 beyond 1024 (512 -> 512 -> 2048 at 16 x 512
// 21.7 / 20.4), and half a us per 512 more that come in before the first product (2048 -> 512 -> 512 there 20.7 / 18.5).  Over
// odd rows at either end the separate layers take longer than their model by more than that (512 -> 512 -> 1024 at 4 x 799 frames
// 16.3 / 21.0), from about 50 groups on (512 -> 512 -> 512 -> 1024 at 1 x 104, 7 groups, 17.0 / 15.4).
// Both sides at 23 sizes of Conformers with and without activations, 16 sizes of 27 kinds of chains and 9 odd ones of 8,
// profiles/merged_launches.txt: what the rule takes runs in 0.56 to 1.00 of the time of separate launches, one case of exactly 256
// workgroups in 1.02 (1024 -> 512 -> 512 at 1 x 4096); what it leaves would have, up to 0.79
// (512 -> 512 -> 512 at 1 x 400, whose stream is shorter than its fixed part says) and over odd rows 0.58 (512 -> 2048 -> 512 at 16 x 399).
bool pw_chain_better(const ConvParams* dw, const ChainOp* op, int n) {
  Plan pl;
  if (!plan(dw, op, n, 256, pl)) return false;
  if (tuning().pw_chain_force) return true;
  if (pl.wgs > 256) return false;
  double blocks = 0.0, apart = dw ? 2.0 : 0.0;
  for (int i = 0; i < n; ++i) {
    double us;
    if (!pw_wide_us(op[i].p, us)) return false;
    blocks += (double)op[i].p.Cin * op[i].p.Cout / (256 * 1024);
    apart += us + 1.2 + (op[i].glu ? 3.2 : 0.0);
  }
  const double out = ((op[n - 1].glu ? op[n - 1].p.Cout / 2 : op[n - 1].p.Cout) - 512) / 512.0, in = (op[0].p.Cin - 512) / 512.0;
  const bool two = n == 2 && pl.MT == 2;
  const ConvParams &f = op[0].p, &e = op[n - 1].p;
  const bool odd = pl.wgs * pl.MT >= 48 && ((!dw && ragged(f.Tin + f.xpad, f.xbs, f.x)) || ragged(e.Tout + e.ypad, e.ybs, e.y));
  const double rows = odd ? 0.0 : two ? (out > 1.0 ? 2.0 * out - 1.0 : out) + 0.5 * in : out;
  const double chain = (pl.MT == 1 ? 7.0 + 2.05 * blocks : 7.5 + 2.2 * blocks) + (dw ? 2.0 : 0.0) + rows;
  return chain < apart;
}

hipError_t launch_pw_chain(const ConvParams* dw, const uint32_t* img, const ChainOp* op, int n, hipStream_t st) {
  Plan pl;
  if (!plan(dw, op, n, compute_units(), pl)) return hipErrorInvalidValue;
  const ConvParams &f = op[0].p, &e = op[n - 1].p;
  ChainParams p{};
  if (dw) {
    p.dw = pl.dw;
    p.dw.img = img;
  } else {
    p.dw.x = f.x; p.dw.xbs = f.xbs; p.dw.xpitch = f.Tin + f.xpad; p.dw.Tin = f.Tin;
    p.xragged = ragged(p.dw.xpitch, f.xbs, f.x);
  }
  p.y = e.y; p.ybs = e.ybs; p.ypitch = e.Tout + e.ypad; p.Tout = e.Tout;
  p.yragged = ragged(p.ypitch, e.ybs, e.y);
  p.n = n;
  const int gpr = (f.Tin + 15) / 16;
  p.tpr = (gpr + pl.MT - 1) / pl.MT;
  p.g_base = gpr / p.tpr;
  p.g_more = gpr % p.tpr;
  p.r_tpr = 1.0f / (float)p.tpr;
  p.wgs = (int)pl.wgs;
  p.per_xcd = (p.wgs + 7) / 8;
  p.buf[0] = pl.buf[0]; p.buf[1] = pl.buf[1];
  p.const_off = pl.const_off; p.table_off = pl.table_off;
  p.rows_off = pl.rows_off; p.row_bytes = pl.row_bytes; p.taps_off = pl.taps_off;
  for (int i = 0; i < n; ++i) {
    const ConvParams& q = op[i].p;
    p.blocks += q.Cin / 512 * (q.Cout / 512);
    p.layer[i] = {q.w, q.bias, q.m, q.s, op[i].table, q.Cin, q.Cout, q.relu, op[i].glu, op[i].glu_m, op[i].glu_s};
  }
  if (!dw) return pl.MT == 1 ? launch_t<1, 0>(p, (size_t)pl.lds, st) : launch_t<2, 0>(p, (size_t)pl.lds, st);
  return pl.MT == 1 ? launch_t<1, 3>(p, (size_t)pl.lds, st) : launch_t<2, 3>(p, (size_t)pl.lds, st);
}

}  // namespace qasr
