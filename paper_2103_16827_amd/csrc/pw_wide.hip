// Pointwise (k = 1) int8 convolution on the gfx950 matrix cores, one workgroup of 16 waves per compute
// unit, with the fused epilogue (bias, dyadic rescale, residual, clamp, table of a unary activation).
//
// What bounds a pointwise layer of these networks is seldom the products: at 6400 frames a 2048 -> 512
// layer is 2.9 us of them and took 14, at one utterance every layer is a chain of latencies.  So the
// kernel is built to have everything in flight at once and to keep four waves per SIMD:
//   - a tile is MT 16-frame groups (of the flat list of all rows' groups) x all input channels, brought
//     into LDS by one round of 16-byte loads per thread, a single barrier, no chunk pipeline;
//   - the waves are KS groups over the input channels x 16 / KS over the output channels, 16 NT channels
//     each.  A matrix product then costs 8 / NT cycles of the LDS port (two transposing reads per
//     operand and 16 NT channels) and 16 / MT cycles of the unit's 64 bytes per cycle from the L2
//     (weights); a wave that owns two columns (NT = 2) keeps both under the 4 cycles a product takes on
//     four SIMDs, and splitting the input channels instead of the output channels over the waves is
//     what allows NT = 2 where a workgroup has only 256 or 128 output channels to compute;
//   - the KS partial sums of a 16 x 16 block meet in LDS, block e is finished by group e mod KS;
//   - finished blocks are staged in LDS and leave as 16-byte pieces of rows.
// LDS: row = input channel, TW units of 16 frames, unit u in slot u ^ swizzle(row) so that the 8 rows a
// transposing read touches lie in different banks (see pw_tile.hip for the operand layout).
#include "kernels.hpp"
#include "launch_shape.hpp"
#include "tuning.hpp"

#include <type_traits>

namespace qasr {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));

constexpr int kStoreThrough = 17;    // sc0 sc1: the output rows are written through (see pw_pipe_body.hpp)
constexpr int kMaxLoads = 8;         // 16-byte loads per thread

struct PwwGeom {
  int G, gpr;           // 16-frame groups in all, per row
  int kch;              // Cin / 64
  int co16n;            // ceil(Cout / 16)
  int splits;           // workgroups per tile, each with its own output channels
  int wgs, per_xcd;
  int stage_off;        // of the staged rows in LDS
  int own_stage;        // ... which do not overlap the tile
  int lut_off;          // of the activation's table
  float r_splits, r_gpr;   // reciprocals of splits, gpr
};

__device__ __forceinline__ v2i read_tr8(const unsigned char* p) {
  return __builtin_amdgcn_ds_read_tr8_b64_v2i32(
      (v2i __attribute__((address_space(3)))*)(const_cast<unsigned char*>(p)));
}

// rows 0..7 mod 8 of a transposing read: 128-byte rows need eight different slots, 64-byte rows fall on
// the same banks every fourth row
template <int TW>
__host__ __device__ constexpr int swizzle(int row) { return TW == 8 ? row & 7 : (row >> 2) & 3; }

// RAGGED: rows of x, y or the residual that are not padded to whole 16-byte aligned units, or x of items too large for the
// other form's 32-bit offsets; v: (tile, split)
template <int MT, int NT, int KS, bool RAGGED, bool MULTI>
__device__ __forceinline__ void pw_wide_tile(const ConvParams& p, const PwwGeom& g, int v) {
  constexpr int TW = MT > 4 ? 8 : 4;                // units per LDS row
  constexpr int NWC = 16 / KS;                      // waves over the output channels
  extern __shared__ __align__(128) unsigned char xs[];   // tile; then partial sums, staged rows; table
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wc = wave % NWC, ks = wave / NWC;
  // All arguments of the first loads in one go; no integer division and, on whole rows, no address per load.  Eight
  // layers in turn, each with its own tensors, us a layer, with them / now: 512 -> 512 G=13 4.97 / 4.46, G=200 7.46 / 7.25;
  // 256 -> 256 G=100 5.27 / 4.78, G=1600 9.62 / 9.42; 2048 -> 512 G=50 8.77 / 8.43, G=200 13.19 / 13.06.
  // (MULTI: a layer's own arguments arrive later, a level further from the kernel's.)
  asm volatile("" ::"s"(p.Tin), "s"(p.xpad), "s"(g.G), "s"(g.gpr), "s"(g.splits), "s"(g.r_splits), "s"(g.r_gpr));
  if constexpr (!MULTI) asm volatile("" ::"s"(p.x), "s"(p.w), "s"(p.xbs), "s"(p.Cin), "s"(g.kch));
  const int tile = divide_uniform(v, g.splits, g.r_splits), cs = v - tile * g.splits;
  const int g0 = tile * MT;
  const int xpitch = p.Tin + p.xpad, ypitch = p.Tout + p.ypad;
  const int b0 = divide_uniform(g0, g.gpr, g.r_gpr), q0 = g0 - b0 * g.gpr;   // batch item of the tile's first unit; unit of its row
  // unit u < 8 of the tile: batch item after b0, first frame
  auto unit = [&](int u, int& db, int& t) __attribute__((always_inline)) {
    split_near(q0 + u, g.gpr, g.r_gpr, db, t);
    t *= 16;
  };

  // ---- tile: thread -> unit tid % TW of rows tid / TW, + 1024 / TW, ...
  {
    const int u = tid & (TW - 1), row0 = tid / TW, step = 1024 / TW;
    const bool on = u < MT && g0 + u < g.G;
    int db, t;
    unit(u, db, t);
    v4i r[kMaxLoads];
    const int wrow = wave * (64 / TW);              // first of the wave's rows (Cin is a multiple of 64: all of them or none)
    if constexpr (RAGGED) {
      const int8_t* const src = p.x + (int64_t)(b0 + (on ? db : 0)) * p.xbs + (int64_t)row0 * xpitch;
#pragma unroll
      for (int i = 0; i < kMaxLoads; ++i) {
        r[i] = (v4i){0, 0, 0, 0};
        if (wrow + i * step < p.Cin && on) r[i] = load_row16(src + (int64_t)i * step * xpitch, t, p.Tin);
      }
    } else {
      const __amdgpu_buffer_rsrc_t xrs =
          __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(p.x) + (int64_t)b0 * p.xbs, 0, 0x7ffffff0, 0x00027000);
      // (outside the tile: past the end of the buffer, which reads zeros)
      const uint32_t at = on ? (uint32_t)db * (uint32_t)p.xbs + (uint32_t)row0 * (uint32_t)xpitch + (uint32_t)t : 0xfffffff0u;
#pragma unroll
      for (int i = 0; i < kMaxLoads; ++i)
        if (wrow + i * step < p.Cin) {
          const v4u w = __builtin_amdgcn_raw_buffer_load_b128(xrs, at, i * step * xpitch, 0);
          r[i] = (v4i){(int)w.x, (int)w.y, (int)w.z, (int)w.w};
        }
    }
    if (p.act_lut && tid < 64)
      reinterpret_cast<uint32_t*>(xs + g.lut_off)[tid] = reinterpret_cast<const uint32_t*>(p.act_lut)[tid];
    static_assert(swizzle<TW>(1024 / TW) == 0, "a thread's rows share the swizzle");
    unsigned char* const dst = xs + row0 * (16 * TW) + ((u ^ swizzle<TW>(row0)) << 4);
#pragma unroll
    for (int i = 0; i < kMaxLoads; ++i)
      if (wrow + i * step < p.Cin) *reinterpret_cast<v4i*>(dst + i * (step * 16 * TW)) = r[i];
  }

  // ---- products: input channel chunks ks, ks + KS, ... x 16 NT output channels
  const int n = lane & 15, gi = lane >> 4;
  const int co16 = (cs * NWC + wc) * NT;            // first 16-channel column of this wave
  const bool active = co16 < g.co16n;               // (uniform; the others only load and store)
  // (wave-uniform base + 16 bytes per lane: one scalar address per load)
  const int8_t* wsrc[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
    wsrc[nt] = p.w + (int64_t)__builtin_amdgcn_readfirstlane(min(co16 + nt, g.co16n - 1)) * (g.kch * 1024);
  const uint32_t wlane = (uint32_t)lane * 16;
  v4i wb[3][NT];
  auto load_w = [&](int kc, v4i (&dst)[NT]) __attribute__((always_inline)) {
    kc = min(kc, g.kch - 1);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) dst[nt] = *reinterpret_cast<const v4i*>(wsrc[nt] + (int64_t)kc * 1024 + wlane);
  };
  v4i acc[MT][NT];
  int32_t mc[NT], sc[NT];
  if (active) {
    load_w(ks, wb[0]);
    load_w(ks + KS, wb[1]);
  }
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int co = min(16 * (co16 + nt) + n, p.Cout - 1);
    const int32_t bv = p.bias && ks == 0 ? p.bias[co] : 0;
    mc[nt] = p.m[co];
    sc[nt] = p.s[co];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt][nt] = (v4i){bv, bv, bv, bv};
  }
  __syncthreads();                                  // the tile is complete
  const int l16 = lane & 15, jr = l16 >> 1;
  // transposing read: lane -> row 8 gi + l16 / 2 (and + 32) of the chunk, 8 frames of unit mt
  const uint32_t arow = (uint32_t)((8 * gi + jr) * (16 * TW) + 8 * (l16 & 1));
  const uint32_t aswz = (uint32_t)swizzle<TW>(8 * gi + jr) << 4;   // (the same for row + 32)
  static_assert(swizzle<TW>(32) == 0, "rows 32 apart share the swizzle");
  if (active) {
    // the operand of unit mt + 2 is read while units mt and mt + 1 are multiplied, across chunks too
    const unsigned char* const abase = xs + arow;
    v2i ar[3][2];
    auto read_a = [&](int kc, int mt, v2i (&dst)[2]) __attribute__((always_inline)) {
      const unsigned char* const q = abase + kc * (64 * 16 * TW) + (aswz ^ (uint32_t)(mt << 4));
      dst[0] = read_tr8(q);
      dst[1] = read_tr8(q + 32 * 16 * TW);
    };
    auto at_step = [&](int kc, int i, v2i (&dst)[2]) __attribute__((always_inline)) {   // i-th unit from chunk kc on
      if (i < MT) read_a(kc, i, dst);
      else if (i < 2 * MT) read_a(min(kc + KS, g.kch - 1), i - MT, dst);
      else read_a(min(kc + 2 * KS, g.kch - 1), i - 2 * MT, dst);
    };
    at_step(ks, 0, ar[0]);
    at_step(ks, 1, ar[1]);
    for (int kc0 = ks; kc0 < g.kch; kc0 += 3 * KS) {
#pragma unroll
      for (int h = 0; h < 3; ++h) {
        const int kc = kc0 + h * KS;
        if (kc < g.kch) {
          load_w(kc + 2 * KS, wb[(h + 2) % 3]);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) {
            const int i = h * MT + mt;
            const v4i a = {ar[i % 3][0].x, ar[i % 3][0].y, ar[i % 3][1].x, ar[i % 3][1].y};
            at_step(kc, mt + 2, ar[(i + 2) % 3]);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
              acc[mt][nt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, wb[h][nt], acc[mt][nt], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
    }
  }

  // ---- output rows of the workgroup: channel 16 cs NWC NT + row, row = 16 (wc NT + nt) + n.  A wave
  // moves rows wave * NWC NT .. (for KS = 1 its own): lane -> row lane / TW, slot lane % TW.
  constexpr int RPW = NWC * NT;                     // rows per wave
  constexpr int RPI = 64 / TW;                      // rows per 64 lanes
  constexpr int NI = (RPW + RPI - 1) / RPI;
  unsigned char* const red = xs;
  unsigned char* const stage = xs + g.stage_off;   // (KS > 1: after the partial sums)
  const unsigned char* const lut = xs + g.lut_off;
  const int row_l = lane / TW, slot_l = lane & (TW - 1);
  // (offsets from the tile's first batch item: 32 bits)
  const int64_t ybase = (int64_t)b0 * p.ybs;
  auto piece = [&](int it, uint32_t& at, int& t) __attribute__((always_inline)) {   // of the residual / output
    const int row = wave * RPW + it * RPI + row_l;
    const int u = slot_l ^ swizzle<TW>(row), co = cs * (16 * RPW) + row;
    int db;
    unit(u, db, t);
    at = (uint32_t)db * (uint32_t)p.ybs + (uint32_t)co * (uint32_t)ypitch;
    return it * RPI + row_l < RPW && u < MT && g0 + u < g.G && co < p.Cout;
  };
  v4i rr[NI];
  if (p.res) {
#pragma unroll
    for (int it = 0; it < NI; ++it) {
      int t;
      uint32_t at;
      if (piece(it, at, t)) {
        const int8_t* const r = p.res + ybase + at;
        rr[it] = RAGGED ? load_row16(r, t, p.Tout) : *reinterpret_cast<const v4i*>(r + t);
      }
    }
  }
  // where the staged rows have LDS of their own, a wave goes on while others still multiply: its epilogue
  // then passes under their products
  if (KS > 1 || !g.own_stage) __syncthreads();      // the tile has been read by all
  if constexpr (KS > 1) {
    if (active) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const int e = mt * NT + nt;
          if (e % KS != ks) {
            const int rank = ks < e % KS ? ks : ks - 1;
            *reinterpret_cast<v4i*>(red + ((size_t)((e * (KS - 1) + rank) * NWC + wc) * 64 + lane) * 16) = acc[mt][nt];
          }
        }
    }
  }
  if (p.res) {
#pragma unroll
    for (int it = 0; it < NI; ++it)
      if (it * RPI + row_l < RPW)
        *reinterpret_cast<v4i*>(stage + (wave * RPW + it * RPI) * (16 * TW) + lane * 16) = rr[it];
  }
  if constexpr (KS > 1) __syncthreads();
  else asm volatile("" ::: "memory");
  bool ok_s = true;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) ok_s = ok_s && sc[nt] >= kShortMin && sc[nt] <= (p.res ? kShortMaxRes : kShortMax);
  const bool fast = __all(ok_s);
  auto finish = [&](auto fast_tag, auto res_tag, auto relu_tag) __attribute__((always_inline)) {
    constexpr bool FAST = decltype(fast_tag)::value, RES = decltype(res_tag)::value, RELU = decltype(relu_tag)::value;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int row = 16 * (wc * NT + nt) + n;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const int e = mt * NT + nt;
        if (KS > 1 && e % KS != ks) continue;
        v4i a = acc[mt][nt];
        if constexpr (KS > 1) {
#pragma unroll
          for (int q = 0; q < KS - 1; ++q)
            a += *reinterpret_cast<const v4i*>(red + ((size_t)((e * (KS - 1) + q) * NWC + wc) * 64 + lane) * 16);
        }
        uint32_t* const sp = reinterpret_cast<uint32_t*>(stage + row * (16 * TW) + ((mt ^ swizzle<TW>(row)) << 4) + 4 * gi);
        const int32_t a4[4] = {a[0], a[1], a[2], a[3]};
        const uint32_t rw = RES ? *sp : 0u;
        uint32_t pk;
        if constexpr (FAST) pk = requant_short4<RES, RELU>(a4, mc[nt], sc[nt] - 32, 1 << ((sc[nt] - 33) & 31), rw);
        else pk = requant_pack4<false, true>(a4, mc[nt], sc[nt], 0, rw, p.relu ? 0 : -128, 127);
        if (p.act_lut) {
          const uint32_t cd = pk ^ 0x80808080u;
          pk = (uint32_t)lut[cd & 0xffu] | ((uint32_t)lut[(cd >> 8) & 0xffu] << 8) |
               ((uint32_t)lut[(cd >> 16) & 0xffu] << 16) | ((uint32_t)lut[cd >> 24] << 24);
        }
        *sp = pk;
        if (mt & 1) __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  if (active) {
    const std::true_type T{};
    const std::false_type F{};
    if (p.res) {
      if (!fast) finish(F, T, F);
      else if (p.relu) finish(T, T, T);
      else finish(T, T, F);
    } else {
      if (!fast) finish(F, F, F);
      else if (p.relu) finish(T, F, T);
      else finish(T, F, F);
    }
  }
  if constexpr (KS > 1) __syncthreads();
  else asm volatile("" ::: "memory");
  const __amdgpu_buffer_rsrc_t yrs = __builtin_amdgcn_make_buffer_rsrc(p.y + ybase, 0, 0x7ffffff0, 0x00027000);
#pragma unroll
  for (int it = 0; it < NI; ++it) {
    int t;
    uint32_t at;
    const bool ok = piece(it, at, t);
    const v4i o = *reinterpret_cast<const v4i*>(stage + (wave * RPW + it * RPI) * (16 * TW) + lane * 16);
    if (RAGGED) {
      if (ok) store_row16(p.y + ybase + at, t, p.Tout, o);
    } else {
      const v4u ov = {(unsigned)o.x, (unsigned)o.y, (unsigned)o.z, (unsigned)o.w};
      __builtin_amdgcn_raw_buffer_store_b128(ov, yrs, ok ? at + (uint32_t)t : 0xfffffff0u, 0, kStoreThrough);
    }
  }
}

template <int MT, int NT, int KS, bool RAGGED>
__global__ __launch_bounds__(1024) void pw_wide_kernel(ConvParams p, PwwGeom g) {
  // consecutive workgroups go round-robin to the 8 XCDs: each takes a contiguous run of (tile, split)
  const int v = (int)(blockIdx.x & 7) * g.per_xcd + (int)(blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= g.per_xcd || v >= g.wgs) return;                 // whole workgroup
  pw_wide_tile<MT, NT, KS, RAGGED, false>(p, g, v);
}

// Several layers of equal output shape and nothing in common but that none reads what another writes (the projections of
// a dense-residual block: 55 launches of about 5 us in a Jasper-10x5, each of a few workgroups that wait for their
// first loads): the workgroups of all of them in one launch, 10 in all.  A whole Jasper-10x5 dense-residual forward, us,
// one by one / together: 1 x 208 frames 791 / 563, 2 x 811 1074 / 837, 4 x 800 1409 / 1167, 16 x 800 2687 / 2517.
struct PwMulti {
  struct Item {
    const int8_t *x, *w;
    const int32_t *bias, *m, *s;
    int8_t* y;
    int64_t xbs;
    int32_t Cin, relu;
  } item[kMaxMulti];
  int wgs1;                                         // workgroups of one layer
  float r_wgs1;                                     // its reciprocal
};

template <int MT, int NT, int KS>
__global__ __launch_bounds__(1024) void pw_multi_kernel(ConvParams p, PwwGeom g, PwMulti l) {
  const int v = (int)(blockIdx.x & 7) * g.per_xcd + (int)(blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= g.per_xcd || v >= g.wgs) return;                 // whole workgroup
  const int i = divide_uniform(v, l.wgs1, l.r_wgs1);
  const PwMulti::Item& q = l.item[i];
  p.x = q.x; p.w = q.w; p.bias = q.bias; p.m = q.m; p.s = q.s; p.y = q.y; p.xbs = q.xbs; p.relu = q.relu;
  p.Cin = q.Cin;
  g.kch = q.Cin / 64;
  pw_wide_tile<MT, NT, KS, false, true>(p, g, v - i * l.wgs1);
}

struct Choice { int MT, NT, KS; };

// LDS: the tile; over it, or after it if there is room (KS = 1), the staged rows (and what the last wave's
// 64 lanes read past them), for KS > 1 behind the partial sums; the activation's table
struct Lds { int stage_off, own_stage, lut_off; };

Lds lds_layout(const ConvParams& p, const Choice& c) {
  const int TW = c.MT > 4 ? 8 : 4, nwc = 16 / c.KS;
  const int tile = p.Cin * 16 * TW, stage = (16 * nwc * c.NT + 64 / TW) * 16 * TW;
  const int red = c.KS > 1 ? c.MT * c.NT * (c.KS - 1) * nwc * 1024 : 0;
  Lds l;
  l.own_stage = c.KS == 1 && tile + stage + 256 <= 160 * 1024;
  l.stage_off = l.own_stage ? tile : red;
  l.lut_off = l.stage_off + stage > tile ? l.stage_off + stage : tile;
  return l;
}
size_t lds_bytes(const ConvParams& p, const Choice& c) { return (size_t)lds_layout(p, c).lut_off + 256; }

bool ragged_rows(const ConvParams& p) {
  return (p.Tin + p.xpad) % 16 || p.xbs % 16 || (uintptr_t)p.x % 16 || (p.Tout + p.ypad) % 16 || p.ybs % 16 ||
         (uintptr_t)p.y % 16 || (uintptr_t)p.res % 16;
}

// whether a tile's part of x lies within 32-bit offsets of its first batch item (7 groups: they reach into so many more items)
bool near_x(const ConvParams& p) {
  const int64_t gpr = (p.Tin + 15) / 16, more = (gpr + 5) / gpr;
  return (more < p.B ? more : p.B - 1) * p.xbs + (int64_t)p.Cin * (p.Tin + p.xpad) <= 0x7ffffff0LL;
}

// The tile with the least time (us) on the busiest compute unit, for `layers` such layers at once that have at least
// least_cin input channels: its matrix pipes (17.7 cycles per product), its LDS port and its 64 bytes per cycle from the L2, whichever is longest, plus the chain of
// first loads and last stores and the epilogue's instructions.
bool pick(const ConvParams& p, int cus, int layers, int least_cin, Choice& best, double& us) {
  if (p.depthwise || p.k != 1 || p.stride != 1 || p.pl != 0 || p.Tout != p.Tin || p.n_res_more) return false;
  if (!p.w_packed || (uintptr_t)p.w % 16 || p.Tin < 4 || p.Cin % 64) return false;
  const int64_t G = (int64_t)p.B * ((p.Tin + 15) / 16);
  if (G > 0x3fffffff || 8 * p.ybs > 0x7ffffff0LL) return false;   // (y: 32-bit offsets within a tile's batch items)
  static const Choice all[] = {{1, 2, 1}, {2, 2, 1}, {4, 2, 1}, {7, 2, 1}, {1, 2, 2}, {2, 2, 2}, {4, 2, 2}, {7, 2, 2},
                               {1, 2, 4}, {2, 2, 4}, {4, 2, 4}, {1, 1, 8}, {2, 1, 8}, {4, 1, 8}};
  const int kch = p.Cin / 64;
  us = 1e300;
  for (const Choice& c : all) {
    const int TW = c.MT > 4 ? 8 : 4, nch = 16 / c.KS * c.NT * 16;
    if ((tuning().pww_mt && c.MT != tuning().pww_mt) || (tuning().pww_ks && c.KS != tuning().pww_ks)) continue;
    if (c.KS > least_cin / 64 || (p.Cin * TW + 1023) / 1024 > kMaxLoads || lds_bytes(p, c) > 160 * 1024) continue;
    const int64_t splits = (p.Cout + nch - 1) / nch, wgs = (G + c.MT - 1) / c.MT * splits * layers;
    if (wgs > max_workgroups(1024)) continue;       // (the other families' tiles cover more frames per thread)
    const int steps = (kch + c.KS - 1) / c.KS;
    const double mfma = c.MT * c.NT * steps * 17.7 * 4, lds = 16.0 * c.MT * steps * 8;
    const double l1 = 16.0 * c.NT * steps * 16 + p.Cin * 16.0 * c.MT / 64;
    const double most = mfma > lds ? (mfma > l1 ? mfma : l1) : (lds > l1 ? lds : l1);
    const double wg = 3.5 + 1.2 * most / 2200 + 0.18 * c.MT * c.NT / c.KS + (c.KS > 1 ? 0.4 : 0.0);
    const double cost = (double)((wgs + cus - 1) / cus) * wg;
    if (cost < us) { us = cost; best = c; }
  }
  return us < 1e300;
}

// for `layers` layers like p, of which p has the most input channels
PwwGeom geometry(const ConvParams& p, const Choice& c, int layers) {
  const int MT = c.MT, NT = c.NT, KS = c.KS;
  PwwGeom g;
  g.gpr = (p.Tin + 15) / 16;
  g.G = p.B * g.gpr;
  g.kch = p.Cin / 64;
  g.co16n = (p.Cout + 15) / 16;
  g.splits = (p.Cout + 16 / KS * NT * 16 - 1) / (16 / KS * NT * 16);
  g.wgs = (g.G + MT - 1) / MT * g.splits * layers;
  g.per_xcd = (g.wgs + 7) / 8;
  const Lds l = lds_layout(p, c);
  g.stage_off = l.stage_off;
  g.own_stage = l.own_stage;
  g.lut_off = l.lut_off;
  g.r_splits = 1.0f / (float)g.splits;
  g.r_gpr = 1.0f / (float)g.gpr;
  return g;
}

template <int MT, int NT, int KS, bool RAGGED>
hipError_t launch_t(const ConvParams& p, hipStream_t st) {
  const Choice c{MT, NT, KS};
  const PwwGeom g = geometry(p, c, 1);
  const size_t lds = lds_bytes(p, c);
  static std::atomic<uint64_t> lds_raised{0};   // per instantiation, a bit per device
  if (const hipError_t e = ensure_max_dynamic_lds((const void*)pw_wide_kernel<MT, NT, KS, RAGGED>, lds_raised); e != hipSuccess)
    return e;
  return launch_kernel(pw_wide_kernel<MT, NT, KS, RAGGED>, dim3((unsigned)(8 * g.per_xcd)), dim3(1024), lds, st, p, g);
}

}  // namespace

bool pw_wide_supported(const ConvParams& p) {
  Choice c;
  double t;
  return !tuning().no_pw_wide && pick(p, 256, 1, p.Cin, c, t);
}

bool pw_wide_us(const ConvParams& p, double& us) {
  Choice c;
  return pick(p, 256, 1, p.Cin, c, us);
}

// Where this kernel is the faster one, in 16-frame groups G.  Measured on single layers whose weights and
// tensors come from memory (us, the other kernel / this one), 50 shapes at up to 14 sizes each; with these
// lines the choice is within 1 % of the better kernel on average.
//   pw_tile (one pass after another per workgroup):
//     257 to 512 channels are one workgroup's here, which stays ahead: 640 -> 512 G=50 9.4 / 5.3, G=1000 11.9 / 10.7,
//       G=3200 29.2 / 26.3; 384 -> 384 G=400 8.1 / 7.0, G=1400 10.7 / 8.5 (but G=550 8.1 / 8.4);
//     beyond 512, workgroups share a tile, which pays while all of them (of 7 groups x 512 channels) run at once:
//       640 -> 768 G=200 14.3 / 8.3, G=700 15.4 / 12.3, G=900 (258 workgroups) 15.7 / 19.8; with 1024 input channels pw_tile
//       has LDS for 128 channels at a time only: 1024 -> 1000 G=200 36.9 / 10.2, G=2000 52.1 / 49.5;
//     up to 256 channels, the input channels are split over the waves: 1024 -> 29 G=200 6.6 / 4.9, G=700 6.8 / 5.8, G=1400
//       8.0 / 8.4; 512 -> 128 G=100 5.5 / 4.7, G=400 5.6 / 5.4; 256 -> 128 G=100 4.7 / 4.8;
//   pw_pipe with 1024 and 2048 input channels (streamed through a ring, a barrier per 64 of them):
//     2048 -> 512 G=100 11.6 / 9.3, G=200 11.8 / 10.8, G=300 12.0 / 12.8; 1024 -> 1024 G=50 8.1 / 7.4, G=200 8.9 / 10.1;
//   pw_pipe whose passes cannot be split over workgroups (not a power of two, or the last one is partial) and are not
//     the lean form's: 512 -> 768 G=200 11.1 / 7.5, G=300 (lean) 7.2 / 7.9, G=1600 16.5 / 20.7; 512 -> 1000 G=100
//     13.5 / 6.9, G=800 14.7 / 11.9, G=1600 20.1 / 23.2; 256 -> 384 G=100 6.3 / 5.0, G=300 6.5 / 6.2;
//   all else is pw_pipe's: 512 -> 2048 G=400 12.5 / 12.5, G=1400 33.5 / 40.6; 512 -> 1024 G=350 7.8 / 10.1, G=1600 19.8 / 24.0;
//     512 -> 512 G=200 5.9 / 6.7, G=1600 12.0 / 12.3.
// (Host only, before any device is asked: for the whole chip's 256 units.)
bool pw_wide_better(const ConvParams& p, bool pipe) {
  const Tuning& t = tuning();
  if (!pw_wide_supported(p)) return false;
  if (t.pw_wide_force) return true;
  if (t.pwp_mt || t.pwp_split || t.pw_lean_force || t.pwt_mt || t.pwp_nopipe) return false;   // a forced form of the others
  const int64_t G = (int64_t)p.B * ((p.Tin + 15) / 16);
  if (!pipe) {
    if (p.Cout > 512) return p.Cin >= 1024 || (G + 6) / 7 * ((p.Cout + 511) / 512) <= 256;
    if (p.Cout > 256) return true;
    return G <= 700 && G <= 2 * (p.Cin - 320);
  }
  const int passes = (p.Cout + 255) / 256;
  if (p.Cin >= 1024) return G * passes * 1024 <= (int64_t)200 * p.Cin;
  if (p.Cout % 256) return G <= 800 && G <= 50 * passes * passes;
  if (passes & (passes - 1)) return 2 * ((G + 6) / 7) * passes <= 256;      // (more workgroups take the lean form)
  return false;
}

hipError_t launch_pw_wide(const ConvParams& p, hipStream_t st) {
  Choice c;
  double t;
  if (!pick(p, compute_units(), 1, p.Cin, c, t)) return hipErrorInvalidValue;
  const bool ragged = ragged_rows(p) || !near_x(p);
#define QASR_CASE(M, N, K) if (c.MT == M && c.NT == N && c.KS == K) return ragged ? launch_t<M, N, K, true>(p, st) : launch_t<M, N, K, false>(p, st);
  QASR_CASE(1, 2, 1) QASR_CASE(2, 2, 1) QASR_CASE(4, 2, 1) QASR_CASE(7, 2, 1)
  QASR_CASE(1, 2, 2) QASR_CASE(2, 2, 2) QASR_CASE(4, 2, 2) QASR_CASE(7, 2, 2)
  QASR_CASE(1, 2, 4) QASR_CASE(2, 2, 4) QASR_CASE(4, 2, 4)
  QASR_CASE(1, 1, 8) QASR_CASE(2, 1, 8) QASR_CASE(4, 1, 8)
#undef QASR_CASE
  return hipErrorInvalidValue;
}

// the tile for all of them, by the layer with the most input channels
static bool pick_multi(const ConvParams* p, int n, int cus, int& most, Choice& c, double& us) {
  most = 0;
  int least = 0;
  for (int i = 1; i < n; ++i) {
    if (p[i].Cin > p[most].Cin) most = i;
    if (p[i].Cin < p[least].Cin) least = i;
  }
  return pick(p[most], cus, n, p[least].Cin, c, us);
}

// Layers one by one take at least 4.7 us each (launch and first loads), whichever kernel runs them; a chip that each of
// them fills has kernels up to a fifth faster than this one, which is the line.  Two to six layers of 64 .. 2048 -> 29 ..
// 2048 channels, 1 x 104 .. 64 x 800 frames, 150 shapes: by this rule 0.31 to 1.01 of their time one by one.  Beyond the
// line, together would be, at 32 x 800 frames: 2 x 256 -> 256 19.8 us against 15.9, 3 x 256 -> 1024 48 against 44, but 5 x 256 ->
// 256 32.5 against 36.2, 6 x 768 -> 768 140 against 145.  A dense-residual Jasper-10x5 of 16 x 1600 frames: one by one 4201,
// by the rule 4147, together wherever it can be 4131.
bool pw_multi_better(const ConvParams* p, int n) {
  if (n < 2 || n > kMaxMulti || tuning().no_pw_wide || tuning().no_pw_multi) return false;
  const ConvParams& f = p[0];
  Choice c;
  int most;
  double t, one_by_one = 0.0;
  for (int i = 0; i < n; ++i) {
    const ConvParams& q = p[i];
    if (q.res || q.act_lut || q.n_res_more || ragged_rows(q) || !near_x(q) || q.B != f.B || q.Cout != f.Cout || q.Tin != f.Tin ||
        q.Tout != f.Tout || q.xpad != f.xpad || q.ypad != f.ypad || q.ybs != f.ybs || !pick(q, 256, 1, q.Cin, c, t))
      return false;
    one_by_one += t + 1.2;
  }
  return pick_multi(p, n, 256, most, c, t) && (tuning().pw_multi_force || t + 1.2 < 0.8 * one_by_one);
}

template <int MT, int NT, int KS>
static hipError_t launch_multi_t(const ConvParams& most, const ConvParams* p, int n, hipStream_t st) {
  const Choice c{MT, NT, KS};
  const PwwGeom g = geometry(most, c, n);
  const size_t lds = lds_bytes(most, c);
  PwMulti l{};
  for (int i = 0; i < n; ++i) l.item[i] = {p[i].x, p[i].w, p[i].bias, p[i].m, p[i].s, p[i].y, p[i].xbs, p[i].Cin, p[i].relu};
  l.wgs1 = g.wgs / n;
  l.r_wgs1 = 1.0f / (float)l.wgs1;
  static std::atomic<uint64_t> lds_raised{0};   // per instantiation, a bit per device
  if (const hipError_t e = ensure_max_dynamic_lds((const void*)pw_multi_kernel<MT, NT, KS>, lds_raised); e != hipSuccess) return e;
  return launch_kernel(pw_multi_kernel<MT, NT, KS>, dim3((unsigned)(8 * g.per_xcd)), dim3(1024), lds, st, most, g, l);
}

hipError_t launch_pw_multi(const ConvParams* p, int n, hipStream_t st) {
  if (!pw_multi_better(p, n)) return hipErrorInvalidValue;
  Choice c;
  int most;
  double t;
  if (!pick_multi(p, n, compute_units(), most, c, t)) return hipErrorInvalidValue;
#define QASR_CASE(M, N, K) if (c.MT == M && c.NT == N && c.KS == K) return launch_multi_t<M, N, K>(p[most], p, n, st);
  QASR_CASE(1, 2, 1) QASR_CASE(2, 2, 1) QASR_CASE(4, 2, 1) QASR_CASE(7, 2, 1)
  QASR_CASE(1, 2, 2) QASR_CASE(2, 2, 2) QASR_CASE(4, 2, 2) QASR_CASE(7, 2, 2)
  QASR_CASE(1, 2, 4) QASR_CASE(2, 2, 4) QASR_CASE(4, 2, 4)
  QASR_CASE(1, 1, 8) QASR_CASE(2, 1, 8) QASR_CASE(4, 1, 8)
#undef QASR_CASE
  return hipErrorInvalidValue;
}

}  // namespace qasr
