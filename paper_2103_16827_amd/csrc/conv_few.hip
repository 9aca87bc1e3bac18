// Dense int8 convolution (k >= 2 taps) for launches of few frames, on the gfx950 int8 matrix cores, with the fused
// epilogue of conv_pipe.hip.
//
// What bounds such a launch is latency and the weights: a 768 -> 768 layer of 25 taps has 14.7 MB, from memory in every
// forward (a Jasper's 322 MB stay in no cache), and a compute unit takes at most 64 bytes per cycle of them.  conv_pipe
// cut the contraction of such layers over workgroups: of 24 us at 2 x 406 frames 7.7 went into handing the partial
// sums over, and its loop took 1000 cycles per step where the weights take 512: three steps ahead are 3000 cycles, the
// latency of memory.  Here
//   - a tile is 16 MT frames x 16 WC NT channels (16, 32, 48 or 64), small enough that there is a workgroup for every unit;
//     narrow ones share a layer's weights out over more units, 48 channels fill one round where 32 begin a second
//     (768 channels, 25 taps, 2 x 406 frames: 22.4 -> 19.1 us; 640, 21 taps 17.7 -> 14.5; 384, 13 taps, 1 x 104 7.1 -> 6.6);
//   - all input channels of the tile are in LDS at once (a layer's 768 channels x 96 frames are 92 KB): one round of
//     loads, one barrier, then 16 waves stream weights with nothing to wait for each other;
//   - they come 8 frames per lane and request, from multiples of 8 on: a unit of the chip takes as long for 4 bytes per lane, and
//     a thread has one unit at most (of 4 frames a 768-channel tile had 1104, and the second round waited for the
//     weights too).  us a layer in chains of six, units of 4 / 8 frames: 1 x 406 frames, 256 channels, 11 taps 6.38 / 5.97, 512, 17 taps
//     9.95 / 9.42, 768, 25 taps 15.7 / 14.9; 2 x 406 7.10 / 6.55, 10.9 / 10.7, 19.8 / 18.8.  From multiples of 4 on, where half of the
//     requests are not aligned, 8.5, 11.7, 16.1; 9.2, 12.3, 19.3.  Rows at odd addresses, 2 x 811 frames of one layer: 256 channels 7.41 / 6.56,
//     640, 21 taps 25.7 / 24.7;
//   - the waves are WC column waves x 16 / WC groups that take the (chunk, tap) steps in turn; a wave has W - 1
//     steps of NT KiB on their way, up to 240 KiB per unit (2 x 48 channels; 144 to 224 the others);
//   - as a wave's stream ends it asks for a dword of each of 64 lines of the weights that this kernel streams next, those
//     that its die's workgroups will read: they come out of memory while a launch ends and the next one begins and
//     brings in its tile, when memory has nothing else to do (a Jasper's layers run at the 2.5 TB/s that their weights come
//     at).  Jasper with dense residuals, 2 x 811 frames: 839 -> 795 us, 732 with the narrow tiles; 1 x 208 566 -> 552 -> 511.
//     A quarter, half, three quarters of the lines 766, 752, 743 us; a dword per 64 bytes 805; asked for before
//     the products, they take the place of lines still to be read: 817;
//   - the groups' sums meet in LDS, a block of 16 x 16 per wave, no workspace.
// us a layer in chains of six, conv_pipe / here: 2 x 406 frames, 256 channels, 11 taps 11.6 / 7.2, 512, 17 taps 16.6 / 10.8,
// 640, 21 taps 20.5 / 17.0; 1 x 104 frames 10.9 / 5.9, 13.3 / 8.7, 14.6 / 10.6; Jasper-10x5 at 1 x 208 input frames 763 -> 551,
// with dense residuals at 2 x 811 1308 -> 1073.  (Before the lines ahead, the narrow tiles and the units of 8 frames.)  What is left: the weights on their way
// out of memory and through the unit's 64 bytes per cycle, and the transposition (about 8 cycles per 64 bytes, 4 us at 768 channels).
// Layouts (operands, packed weights, the 4 x 4 transposition, 80-byte rows) are those of conv_pipe.hip.
#include "kernels.hpp"
#include "launch_shape.hpp"
#include "tuning.hpp"
#include "vmem.hpp"

#include <cmath>
#include <type_traits>

namespace qasr {

namespace {

constexpr int kXS = 80;       // LDS row pitch in bytes: 64 channels + 16 pad
constexpr int kLds = 160 * 1024;

// Weights that a later launch will stream, to be in each die's L2 by then: for die x `runs` runs of lines[x] 128-byte lines, the
// first at w + off[x], `stride` bytes apart.  None: no runs, but w can be read all the same.
struct Ahead {
  const int8_t* w;
  uint32_t runs, stride;
  uint32_t off[8], lines[8];
};

struct FewGeom {
  int n_tt;           // frame tiles per batch item
  int rows;           // LDS rows per chunk (input frames incl. halo, rounded to 8)
  int kchunks;        // Cin / 64
  int co16n;          // ceil(Cout / 16)
  int tiles, per_xcd;
  int units;          // transposition units (8 frames x 16 channels): kchunks * rows / 2, one per thread at most
  int jstep;          // KG / kchunks
  float r_nbt, r_tt, r_rows;   // reciprocals of B * n_tt, n_tt, rows / 2
  Ahead ahead;
};

static_assert(kLds / kXS / 2 <= 1024, "a tile whose rows fit LDS has a unit per thread at most");

// steps of weights on their way and multiplied (registers)
template <int MT, int NT> struct Ring { static constexpr int W = NT == 1 ? 12 : NT == 3 ? (MT == 2 ? 6 : 4) : MT == 4 ? 6 : 8; };
// parts in which the sums meet: all of them, 16 MT NT KiB, have to fit LDS
constexpr int meetings(int MT, int NT) { return 16 * MT * NT > 152 ? 2 : 1; }

// 16 MT frames x 16 WC NT channels: WC column waves of NT columns each
template <int MT, int WC, int NT>
__global__ __launch_bounds__(1024) void conv_few_kernel(ConvParams p, FewGeom g) {
  extern __shared__ __align__(16) unsigned char xs[];   // [kchunks][rows][kXS]; then the partial sums
  constexpr int KG = 16 / WC, W = Ring<MT, NT>::W, AR = 4;
  static_assert(MT * W % AR == 0, "rings");
  asm volatile("" ::"s"(p.x), "s"(p.w), "s"(p.xbs), "s"(p.B), "s"(p.Tin), "s"(p.k), "s"(p.stride), "s"(p.dil), "s"(p.pl), "s"(p.xpad),
               "s"(g.n_tt), "s"(g.rows), "s"(g.kchunks), "s"(g.co16n), "s"(g.tiles), "s"(g.per_xcd), "s"(g.units), "s"(g.jstep), "s"(g.r_nbt),
               "s"(g.r_tt), "s"(g.r_rows));
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wc = wave % WC, kg = wave / WC;
  const int n = lane & 15, gi = lane >> 4;
  // channel tile first, then batch item, then frame tile; XCD x takes a contiguous run of that order (conv_pipe.hip)
  const int v = (int)(blockIdx.x & 7) * g.per_xcd + (int)(blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= g.per_xcd || v >= g.tiles) return;               // whole workgroup
  const int nbt = p.B * g.n_tt;                     // (workgroups: < 2^22)
  const int co_tile = divide_uniform24(v, nbt, g.r_nbt), bt = v - co_tile * nbt;
  const int b = divide_uniform24(bt, g.n_tt, g.r_tt), t0 = (bt - b * g.n_tt) * (16 * MT);
  const int f0 = t0 * p.stride - p.pl;              // first input frame the tile reads
  const int fa = f0 & ~7, foff = f0 - fa;           // rounded down to eight frames (also if negative)
  const int xpitch = p.Tin + p.xpad;

  // ---- weights: steps kg, kg + KG, ... of the flat list (tap, chunk), in the order of the packed weights: together
  // the groups read runs of kchunks KiB
  const int Q = g.kchunks * p.k;
  const int steps = (Q - kg + KG - 1) / KG;         // (may be 0)
  // (chunk and tap of a step, advanced by KG steps)
  const int jstep = g.jstep, kstep = KG - jstep * g.kchunks;
  struct At { int kc, j; };
  At first{kg, 0};
  while (first.kc >= g.kchunks) { first.kc -= g.kchunks; ++first.j; }   // (uniform)
  auto advance = [&](At& a) __attribute__((always_inline)) {
    a.kc += kstep;
    a.j += jstep;
    if (a.kc >= g.kchunks) { a.kc -= g.kchunks; ++a.j; }
  };
  const int col = (co_tile * WC + wc) * NT;         // first 16-channel column of the wave
  uint32_t woff[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) woff[nt] = (uint32_t)((min(col + nt, g.co16n - 1) * g.kchunks * 64 + lane) * 16);
  v4i wb[W][NT];
  At wat = first;
  auto load_w = [&](v4i (&dst)[NT]) __attribute__((always_inline)) {
    const int8_t* const base = p.w + (int64_t)(wat.j * g.co16n * g.kchunks + wat.kc) * 1024;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) dst[nt] = gload16(base, woff[nt]);
    advance(wat);
  };

  // ---- activations: unit = frames 8 fq .. + 8 of the 16 channels of column group cg of chunk kc (conv_pipe.hip), one per thread
  // at most; unit index = (kc * 4 + cg) * (rows / 8) + fq.  16 lanes with consecutive fq write rows 640 bytes apart, which is two
  // of 16 sets of banks: they write their eight rows in an order turned by (fq >> 1) & 7, within the half by the
  // byte selectors and between the halves by a swap, and cover all banks.
  const int nfq = g.rows >> 3;
  const int8_t* const xb = p.x + (int64_t)b * p.xbs;
  v2i xr[4][4];
  // (unit < 2^16: the estimate of unit / (rows / 2) is off by one at most)
  const int uu = min(tid, g.units - 1), half_rows = g.rows >> 1;
  int u_kc = (int)((float)uu * g.r_rows), u_r = uu - u_kc * half_rows;
  if (u_r < 0) { --u_kc; u_r += half_rows; }
  if (u_r >= half_rows) { ++u_kc; u_r -= half_rows; }
  const int u_cg = (u_r >= nfq ? 1 : 0) + (u_r >= 2 * nfq ? 1 : 0) + (u_r >= 3 * nfq ? 1 : 0);
  const int u_fq = u_r - u_cg * nfq, u_f = fa + 8 * u_fq;
  // (what lies over a row's end is loaded from inside the row and moved, what lies outside dropped; rows shorter than eight frames are
  // loaded to their end, from the row before on, the first ones from their start)
  int u_at = max(min(u_f, p.Tin - 8), min(p.Tin - 8, 0));
  if (u_kc + u_cg == 0) u_at = max(u_at, 0);
  if (64 * wave < g.units) {                        // (uniform)
    const uint32_t off = (uint32_t)((64 * u_kc + 8 * u_cg) * xpitch + u_at);   // (Cin x pitch < 2^31)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) xr[i][e] = gload8(xb + (int64_t)(4 * ((i & 1) + 8 * (i >> 1)) + e) * xpitch, off);
  }
  // byte selectors: a half's frames where they lie in the eight, zeros for those that there are not
  const bool swap = (u_fq >> 3) & 1;
  uint32_t half[2];
  {
    const int there = u_f >= 0 ? min(p.Tin - u_f, 8) : 0;           // (u_f is a multiple of 8)
    const uint64_t kept = there > 0 ? ~0ull >> (64 - 8 * there) : 0ull;
    const uint32_t lo = (uint32_t)kept, hi = (uint32_t)(kept >> 32), up = 0x01010101u * (uint32_t)(u_f - u_at);
    const uint32_t s_lo = ((0x03020100u + up) & lo) | (0x0c0c0c0cu & ~lo), s_hi = ((0x07060504u + up) & hi) | (0x0c0c0c0cu & ~hi);
    half[0] = swap ? s_hi : s_lo;
    half[1] = swap ? s_lo : s_hi;
  }
#pragma unroll
  for (int q = 0; q < W - 1; ++q)
    if (q < steps) load_w(wb[q]);
  wait_vm_dyn(min(steps, W - 1) * NT);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) tie(xr[i][e]);
  if (tid < g.units) {
    const int rot = (u_fq >> 1) & 3;
    const uint32_t f0s = rot, f1s = (rot + 1) & 3, f2s = (rot + 2) & 3, f3s = (rot + 3) & 3;
    const uint32_t sel_lo = f0s | ((4 + f0s) << 8) | (f1s << 16) | ((4 + f1s) << 24);
    const uint32_t sel_hi = f2s | ((4 + f2s) << 8) | (f3s << 16) | ((4 + f3s) << 24);
    unsigned char* const unit = xs + (u_kc * g.rows + 8 * u_fq) * kXS + 16 * u_cg;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      unsigned char* const dst = unit + ((h != 0) != swap ? 4 * kXS : 0);
      uint32_t c[4][4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        uint32_t r[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = __builtin_amdgcn_perm((uint32_t)xr[i][e].y, (uint32_t)xr[i][e].x, half[h]);
        const uint32_t lo01 = __builtin_amdgcn_perm(r[1], r[0], sel_lo), hi01 = __builtin_amdgcn_perm(r[1], r[0], sel_hi);
        const uint32_t lo23 = __builtin_amdgcn_perm(r[3], r[2], sel_lo), hi23 = __builtin_amdgcn_perm(r[3], r[2], sel_hi);
        c[i][0] = __builtin_amdgcn_perm(lo23, lo01, 0x05040100u);
        c[i][1] = __builtin_amdgcn_perm(lo23, lo01, 0x07060302u);
        c[i][2] = __builtin_amdgcn_perm(hi23, hi01, 0x05040100u);
        c[i][3] = __builtin_amdgcn_perm(hi23, hi01, 0x07060302u);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
        *reinterpret_cast<v4i*>(dst + ((e + rot) & 3) * kXS) = (v4i){(int)c[0][e], (int)c[1][e], (int)c[2][e], (int)c[3][e]};
    }
  }
  v4i acc[MT][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = (v4i){0, 0, 0, 0};
  __syncthreads();                                  // the tile is complete

  // ---- a lane's line of the weights that come after these (the lines in turn over the die's workgroups, so that each wave asks
  // once at most; past the last one, or if there are none: the first)
  const int8_t* line_ahead = g.ahead.w;
  {
    const int die = (int)(blockIdx.x & 7), wgs = min(g.per_xcd, g.tiles - die * g.per_xcd);
    const uint32_t lines = g.ahead.lines[die], L = (blockIdx.x >> 3) + (uint32_t)(wgs * tid);
    if (L < g.ahead.runs * lines) {
      const float r = (float)L / (float)lines;
      uint32_t run = (uint32_t)r;
      uint32_t at = L - run * lines;
      if ((int32_t)at < 0) { --run; at += lines; }
      if (at >= lines) { ++run; at -= lines; }
      line_ahead = g.ahead.w + (g.ahead.off[die] + run * g.ahead.stride + at * 128);
    }
  }
  // the constants of the block this wave finishes
  constexpr int NB = WC * MT * NT;
  static_assert(NB <= 16, "a block per wave");
  const int e_wc = wave / (MT * NT), e_mt = wave % (MT * NT) / NT, e_nt = wave % NT;
  const int co = ((co_tile * WC + e_wc) * NT + e_nt) * 16 + n, cl = min(co, p.Cout - 1);
  int32_t mc = 0, sc = 33, bv = 0, line = 0;
  if (wave < NB) {
    gload4_into(mc, p.m + cl);
    gload4_into(sc, p.s + cl);
    gload4_into(bv, (p.bias ? p.bias : p.m) + cl);
  }

  // ---- products; operand of item i = unit i % MT of the wave's step i / MT, AR - 1 of them on their way
  const uint32_t abase = (uint32_t)((foff + n * p.stride) * kXS + 16 * gi);
  At aat = first;
  v4i ar[AR];
  auto read_a = [&](int mt, v4i& dst) __attribute__((always_inline)) {
    const int row = aat.kc * g.rows + min(aat.j, p.k - 1) * p.dil + 16 * mt * p.stride;   // (past the end: not used)
    dst = *reinterpret_cast<const v4i*>(xs + abase + (uint32_t)(row * kXS));
  };
#pragma unroll
  for (int i = 0; i < AR - 1; ++i) {
    if (i > 0 && i % MT == 0) advance(aat);
    read_a(i % MT, ar[i]);
  }
  int left = steps;
  const bool whole = steps % W == 0;                // the last round asks for a step's weights after the line
  auto step = [&](auto slot_tag) __attribute__((always_inline)) {
    constexpr int q = decltype(slot_tag)::value;
    if (left >= W - 1) wait_vm<(W - 2) * NT>();
    else if (whole) wait_vm<0>();
    else wait_vm<1>();                              // (nothing but the line is younger than the rest of the stream: all of that)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) tie(wb[q][nt]);
    if (left >= W) load_w(wb[(q + W - 1) % W]);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      constexpr int i0 = q * MT;
      if ((mt + AR - 1) % MT == 0) advance(aat);
      read_a((mt + AR - 1) % MT, ar[(i0 + mt + AR - 1) % AR]);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
        acc[mt][nt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ar[(i0 + mt) % AR], wb[q][nt], acc[mt][nt], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    return --left > 0;
  };
  auto round = [&](auto self, auto slot_tag) __attribute__((always_inline)) -> bool {
    constexpr int q = decltype(slot_tag)::value;
    if constexpr (q < W) return step(slot_tag) && self(self, std::integral_constant<int, q + 1>{});
    else return true;
  };
  do {
    if (left <= W) gload4_into(line, line_ahead);   // (once, in the last round)
  } while (left > 0 && round(round, std::integral_constant<int, 0>{}));
  wait_vm<1>();
#pragma unroll
  for (int q = 0; q < W; ++q)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) tie(wb[q][nt]);
  tie(mc);
  tie(sc);
  tie(bv);

  // ---- block e = (column wave, frame group, column) is finished by wave e
  __syncthreads();                                  // the tile has been read by all
  constexpr int H = meetings(MT, NT), MH = MT / H;
  static_assert(MT % H == 0, "parts");
  v4i* const red = reinterpret_cast<v4i*>(xs);      // [column wave][frame group][column][group][lane]
  v4i a = {0, 0, 0, 0};
#pragma unroll
  for (int h = 0; h < H; ++h) {
    if (h) __syncthreads();
#pragma unroll
    for (int mt = h * MH; mt < (h + 1) * MH; ++mt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) red[(((wc * MH + mt - h * MH) * NT + nt) * KG + kg) * 64 + lane] = acc[mt][nt];
    __syncthreads();
    if (wave < NB && e_mt / MH == h) {
      const int at = ((e_wc * MH + e_mt - h * MH) * NT + e_nt) * KG;
#pragma unroll
      for (int q = 0; q < KG; ++q) a += red[(at + q) * 64 + lane];
    }
  }
  if (wave >= NB) {
    wait_vm<0>();
    tie(line);
    return;
  }

  // lane (n, gi) holds frames t .. + 4 of channel co
  const int t = t0 + 16 * e_mt + 4 * gi;
  if (co < p.Cout && t < p.Tout) {
    const int trow = p.Tout + p.ypad;                 // (pad bytes may be written)
    const int64_t orow = (int64_t)b * p.ybs + (int64_t)co * trow;
    if (!p.bias) bv = 0;
    int32_t o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = dyadic_rescale(a[i] + bv, mc, sc);
    if (p.res) {                                      // residual operands, all on their way at once
      uint32_t d[1 + kMaxMoreRes];
      const int at = min(t, trow - 4), shr = 8 * (t - at);
      d[0] = load_u32(p.res + orow + at);
#pragma unroll
      for (int r = 0; r < kMaxMoreRes; ++r)
        if (r < p.n_res_more) d[r + 1] = load_u32(p.res_more[r] + orow + at);
#pragma unroll
      for (int r = 0; r <= kMaxMoreRes; ++r)
        if (r <= p.n_res_more) {
          const uint32_t w = d[r] >> shr;
#pragma unroll
          for (int i = 0; i < 4; ++i) o[i] += (int32_t)(int8_t)(w >> (8 * i));
        }
    }
    const int lo = p.relu ? 0 : -128;
    uint32_t pk = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) pk |= (uint32_t)(clamp_i8(o[i], lo) & 0xff) << (8 * i);
    store_row_u32(p.y + orow, t, trow, pk);
  }
  wait_vm<0>();
  tie(line);
}

int lds_rows(const ConvParams& p, int TM) { return (((TM - 1) * p.stride + p.dil * (p.k - 1) + 1 + 7) + 7) & ~7; }

size_t lds_bytes(const ConvParams& p, const FewTile& c) {
  const size_t tile = (size_t)(p.Cin / 64) * lds_rows(p, 16 * c.MT) * kXS, sums = (size_t)16 * c.MT * c.NT * 1024 / meetings(c.MT, c.NT);
  return tile > sums ? tile : sums;
}

int64_t workgroups(const ConvParams& p, const FewTile& c) {
  const int C = 16 * c.WC * c.NT;
  return (int64_t)p.B * ((p.Tout + 16 * c.MT - 1) / (16 * c.MT)) * ((p.Cout + C - 1) / C);
}

// what the kernel takes for granted of a layer's tile
bool fits(const ConvParams& p, const FewTile& c) {
  return lds_bytes(p, c) <= (size_t)kLds && (p.Cin / 64) * lds_rows(p, 16 * c.MT) < 65536 && workgroups(p, c) < (1 << 22) - 8;
}

bool supported(const ConvParams& p) {
  if (p.depthwise || p.Cin % 64 || !p.w_packed || p.k < 2 || p.Cout < 64 || p.Tin < 4 || p.Tout < 4 || (uintptr_t)p.w % 16) return false;
  if ((int64_t)p.k * ((p.Cout + 15) / 16) * (p.Cin / 64) * 1024 > 0x7fffffffLL) return false;   // 32-bit offsets
  return (int64_t)p.Cin * (p.Tin + p.xpad) <= 0x7fffffffLL;
}

// The tile with the least time, in cycles: a launch, and on the busiest compute unit for each of its workgroups the
// activations it transposes (64 bytes at a time), its steps (the weights of all its columns, or its products) and its
// last stores; of single columns each operand read serves one product.  Every tile timed beside the choice, chains of six
// layers of 256 .. 768 channels, 11 .. 25 taps, 52 .. 3200 frames (50 shapes, profiles/dense_tile_choice.txt): it is 0.3 % from the best on average
// and 1.6 % at worst; the choice between this kernel and conv_pipe, over 60 shapes to 12800 frames, 0.3 % and 4.1 % (768 channels, 4 x 400
// frames, 35.6 us for 34.1; with 7 cycles per 64 bytes transposed it was up to 17 %, with 10.7, of the units of 4 frames, 14 % off).
// (Constants fitted to those chains alone, whose weights stay in the memory-side cache, make whole networks slower: 732 -> 741.)
bool pick(const ConvParams& p, FewTile& best, double& cycles) {
  if (!supported(p)) return false;
  cycles = 1e300;
  static const FewTile columns[] = {{0, 1, 1}, {0, 1, 2}, {0, 1, 3}, {0, 2, 2}};
  for (FewTile c : columns)
    for (int MT = 1; MT <= 4; ++MT) {
      c.MT = MT;
      if ((tuning().cf_mt && MT != tuning().cf_mt) || (tuning().cf_wc && c.WC != tuning().cf_wc) || (tuning().cf_nt && c.NT != tuning().cf_nt)) continue;
      if (!fits(p, c)) continue;
      const int C = c.WC * c.NT;
      const double step = fmax(C * fmax(6.4 * MT, 24.8), c.NT == 1 ? 12.0 * MT : 0.0);
      const double wg = 3460.0 + 157.5 * MT * C + (double)(p.Cin / 64) * p.k * step + 8.5 * (p.Cin / 64) * lds_rows(p, 16 * MT);
      const double cost = 6300.0 + (double)((workgroups(p, c) + 255) / 256) * wg;
      if (cost < cycles) { cycles = cost; best = c; }
    }
  return cycles < 1e300;
}

void geometry(const ConvParams& p, const FewTile& c, FewGeom& g) {
  g.n_tt = (p.Tout + 16 * c.MT - 1) / (16 * c.MT);
  g.rows = lds_rows(p, 16 * c.MT);
  g.kchunks = p.Cin / 64;
  g.co16n = (p.Cout + 15) / 16;
  g.tiles = (int)workgroups(p, c);
  g.per_xcd = (g.tiles + 7) / 8;
  g.units = g.kchunks * g.rows / 2;
  g.jstep = 16 / c.WC / g.kchunks;
  g.r_nbt = 1.0f / (float)(p.B * g.n_tt);
  g.r_tt = 1.0f / (float)g.n_tt;
  g.r_rows = 2.0f / (float)g.rows;
}

// what the launch of `next` will stream: a die's run of its tiles, channel tile first, spans some of its channel tiles
Ahead weights_of(const ConvParams& next, const FewTile& c) {
  Ahead a{};
  FewGeom g;
  geometry(next, c, g);
  const int nbt = next.B * g.n_tt, column = g.kchunks * 8;     // (lines of 16 channels and a tap)
  a.w = next.w;
  a.runs = (uint32_t)next.k;
  a.stride = (uint32_t)(g.co16n * column * 128);
  for (int x = 0; x < 8; ++x) {
    const int lo = x * g.per_xcd, hi = lo + g.per_xcd < g.tiles ? lo + g.per_xcd : g.tiles;
    if (lo >= hi) continue;
    const int C = c.WC * c.NT, from = lo / nbt * C, to = ((hi - 1) / nbt + 1) * C;
    a.off[x] = (uint32_t)(from * column * 128);
    a.lines[x] = (uint32_t)(((to < g.co16n ? to : g.co16n) - from) * column);
  }
  return a;
}

template <int MT, int WC, int NT>
hipError_t launch_t(const ConvParams& p, const Ahead& ahead, hipStream_t st) {
  const FewTile c{MT, WC, NT};
  FewGeom g;
  geometry(p, c, g);
  g.ahead = ahead;
  if (!g.ahead.w) g.ahead.w = p.w;
  static std::atomic<uint64_t> lds_raised{0};   // per instantiation, a bit per device
  if (const hipError_t e = ensure_max_dynamic_lds((const void*)conv_few_kernel<MT, WC, NT>, lds_raised); e != hipSuccess) return e;
  return launch_kernel(conv_few_kernel<MT, WC, NT>, dim3((unsigned)(8 * g.per_xcd)), dim3(1024), lds_bytes(p, c), st, p, g);
}

}  // namespace

bool conv_few_cycles(const ConvParams& p, FewTile& tile, double& cycles) {
  return !tuning().no_conv_few && pick(p, tile, cycles);
}

hipError_t launch_conv_few(const ConvParams& p, const FewTile& c, const ConvParams* next, const FewTile& next_tile, hipStream_t st) {
  if (!supported(p) || !fits(p, c)) return hipErrorInvalidValue;
  const Ahead ahead = next && supported(*next) && fits(*next, next_tile) ? weights_of(*next, next_tile) : Ahead{};
#define QASR_CASE(C, T) \
  if (c.WC == C && c.NT == T) \
    return c.MT == 1 ? launch_t<1, C, T>(p, ahead, st) : c.MT == 2 ? launch_t<2, C, T>(p, ahead, st) : c.MT == 3 ? launch_t<3, C, T>(p, ahead, st) : launch_t<4, C, T>(p, ahead, st);
  QASR_CASE(1, 1) QASR_CASE(1, 2) QASR_CASE(1, 3) QASR_CASE(2, 2)
#undef QASR_CASE
  return hipErrorInvalidValue;
}

}  // namespace qasr
