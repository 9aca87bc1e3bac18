// Separable module, depthwise and pointwise layer in one kernel (gfx950).
//
//     h[ci, t] = act(clamp(rescale(sum_j x[ci, t - pl + j dil] wd[ci, j])))          (int8, in LDS only)
//     y[co, t] = clamp(rescale(bias + sum_ci W[co, ci] h[ci, t]) + residual)
//
// As two launches a module costs two launch gaps and two chains of first loads (about 5 us each, most
// of the 8 us a depthwise and the 14 us a pointwise layer of 512 channels take at batch 32), and h
// travels to memory and back.  Here a workgroup of 16 waves owns up to MT 16-frame groups of one batch
// item and all channels of them: every wave computes the depthwise layer of Cin / 16 channels for those
// frames into the LDS tile that the pointwise half multiplies from.  Only x is read twice (the halo
// of k - 1 frames between neighbouring tiles, out of the L2).
//
// Depthwise half.  v_mfma_i32_4x4x4_16b_i8 is 16 independent 4 x 4 x 4 products: block = channel.
// With a 4-row Toeplitz operand A[m, kappa] = w[kappa - m - r] (4 kappa per step) and
// B[kappa, n] = x[4 n + kappa], block b, column n, row m yields frame 16 q + 4 n + m of channel b: a lane
// ends with 4 consecutive frames of one channel, ready to be packed.  Against the 16-row form of
// dw_pipe.hip the operand is 4 instead of 16 bytes per tap, small enough to be made from a channel's row of weights
// in LDS by one byte permutation per dword, and a tile of a few groups wastes no columns (16 x 16 x 64 wants 256 frames of a
// channel).  (The operand as a prebuilt image is four times the bytes through the address path: 15x5, 32 x 1600 1208 -> 1172 us.)  It runs
// at 10 cycles per product, (k + 3) / 4 products per 16 frames of 16 channels: at k = 75 that is 5 us
// for 512 channels x 112 frames.  The window dwords are read one by one: a 16-byte LDS read at a 4-byte aligned
// address measured 59 cycles against 16.
//
// Pointwise half: as pw_pipe_body.hpp (transposing LDS reads, packed weights straight from L2), one
// pass of 16 NT channels per wave, compiler-visible loads.
//
// Two kernels: launches of few frames are bound by what a workgroup loads (sep_small_kernel), the others by their
// products (sep_kernel).  Graph replays of QuartzNet-15x5, before sep_small_kernel, place() below and the shorter
// beginnings of the pointwise kernels / with them, projections apart: 1 x 1237 frames 628 / 561 us, 32 x 1600 1163 / 1135;
// 10x5, 8 x 1104 503 / 485.
//
// A block's residual projection, which reads what its first pair reads, runs in the pair's launch: workgroups of
// their own take x itself for the tile and go on with the pointwise half.  At few frames they find units that the pair
// leaves free, at many they start on each unit as it finishes; either way a launch and its chain of first loads
// disappear.  Apart / together: 15x5, 1 x 1237 561 / 484 us, 32 x 1600 1135 / 1102, 64 x 1600 2146 / 2115; 10x5, 8 x 1104
// 485 / 447 (inputs that change from pass to pass, all three steps: 15x5, 32 x 1600 1326 -> 1230).
#pragma once
#include "sep.hpp"
#include "vmem.hpp"

#include <type_traits>

namespace qasr {
namespace sep {

typedef unsigned v4u __attribute__((ext_vector_type(4)));

constexpr int kStoreThrough = 17;    // sc0 sc1: the output rows are written through (see pw_pipe_body.hpp)
constexpr int kWaves = 16;           // 4 per SIMD: each phase's latencies pass under another wave's products
constexpr int kMaxUnits = 15;        // chunks per row in LDS: 16 rows are at most four 64-lane loads

__device__ __forceinline__ v2i read_tr8(const unsigned char* p) {
  return __builtin_amdgcn_ds_read_tr8_b64_v2i32(
      (v2i __attribute__((address_space(3)))*)(const_cast<unsigned char*>(p)));
}

constexpr uint32_t kNone = 0xfffffff0u;             // an offset beyond every buffer's range: the load returns zeros

// Rows of x come as 16-frame chunks, zeros where a row has none, one request per 64 chunks, with no branch around it and nothing
// merged into its register: for `r = 0; if (there) r = load` the compiler moved registers, and to do that waited for all
// that was on its way, a round trip to memory before the pointwise half's weights were even asked for.  Chunks that
// do not exist are out of a buffer's range and come back as zeros; ragged rows (no alignment, no pad) are read past their
// end, the tensor's last ones from inside it.  The frames past a row's end are cleared in LDS, by the tiles that have any.
//
// 16 bytes at off from `rows`, the first of C rows; `tail`: they are the tensor's last
template <int C, bool RAGGED>
__device__ __forceinline__ uint32_t last_start(const DwParams& p, bool tail) {
  return RAGGED && tail ? (uint32_t)((C - 1) * p.xpitch + p.Tin - 16) : kNone;
}
template <int C, bool RAGGED>
__device__ __forceinline__ v4i load_chunk(const DwParams& p, const int8_t* rows, bool tail, uint32_t off, uint32_t step) {
  if constexpr (RAGGED) {
    const uint32_t o = off == kNone ? 0u : min(off + step, last_start<C, RAGGED>(p, tail));
    return *reinterpret_cast<const unaligned_chunk16*>(rows + o);
  } else {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(rows), 0, C * p.xpitch, 0x00027000);
    return __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rs, off, step, 0));
  }
}
// what it brought as it goes to LDS
template <int C, bool RAGGED>
__device__ __forceinline__ v4i whole_chunk(const DwParams& p, bool tail, uint32_t off, uint32_t step, v4i v) {
  if constexpr (RAGGED) {
    const uint32_t end = last_start<C, RAGGED>(p, tail);
    if (__any(off != kNone && off + step > end)) {  // (the tensor's last tile) moved down; zeros come in
      const int n = off != kNone && off + step > end ? (int)(off + step - end) : 0;
      if (n & 8) v = (v4i){v[2], v[3], 0, 0};
      if (n & 4) v = (v4i){v[1], v[2], v[3], 0};
      v4i r;
#pragma unroll
      for (int i = 0; i < 4; ++i) r[i] = (int)__builtin_amdgcn_alignbyte(i < 3 ? (uint32_t)v[i + 1] : 0u, (uint32_t)v[i], (uint32_t)n & 3u);
      v = r;
    }
    if (off == kNone) v = (v4i){0, 0, 0, 0};
  }
  return v;
}
// C rows in LDS, `pitch` bytes apart, whose first chunk starts at frame 16 c0
template <int C>
__device__ __forceinline__ void clear_past_end(const DwParams& p, unsigned char* rows, int pitch, int c0, int lane) {
  const int u = (p.Tin >> 4) - c0;                  // the chunk a row ends in
  if ((p.Tin & 15) && (uint32_t)(16 * u) < (uint32_t)pitch && lane < C) {   // (uniform but for the lane)
    asm volatile("" ::: "memory");                  // (lanes read what other lanes of the wave wrote: LDS is in order)
    v4i* const q = reinterpret_cast<v4i*>(rows + lane * pitch + 16 * u);
    *q = keep_bytes(*q, p.Tin & 15);
  }
}

// 64-lane loads that bring in C rows: at most (MT + NA + 1) | 1 chunks each (units_of: the first chunk starts up to
// 15 frames early, NA quads hold up to 16 NA - 3 frames of taps)
constexpr int row_loads(int C, int MT, int NA) {
  const int u = (MT + NA + 1) | 1;
  return (C * (u < kMaxUnits ? u : kMaxUnits) + 63) / 64;
}

// 16-byte units per row in LDS of the small kernel (odd: 16 rows then start in different banks) and the lanes that bring a row in
constexpr int row_units(int MT, int NA) { return (MT + NA + 1) | 1; }
constexpr int max_row_lanes_log2(int MT, int NA) { return MT + NA + 1 > 8 ? 4 : 3; }

// bytes of a wave's row buffer: 16 rows and what the windows of the last row read past it, at least
// the 16 x 128 bytes of the output staging; of the small kernel's: all C rows, at least
// two 16 x 16 blocks of sums
__host__ __device__ inline int row_bytes(int units, int MT, int NA) {
  const int rows = 15 * 16 * units + 16 * (MT + NA) + 32;
  return ((rows > 2048 ? rows : 2048) + 15) & ~15;
}
__host__ __device__ constexpr inline int small_row_bytes(int C, int units, int MT, int NA) {
  const int rows = (C - 1) * 16 * units + 16 * (MT + NA) + 32;
  return ((rows > 2048 ? rows : 2048) + 15) & ~15;
}

// The workgroup's tile and output channels.  Every scalar instruction costs a unit 16 cycles for 16 waves, the first loads wait
// for all of these: no division, no selection between the two layers' arguments.  All arguments are read first, in one
// go: asked for where they are used, they were a dozen dependent scalar loads.
struct Place { int b, g0, gn, cs; };
// two neighbours of the arguments (an asm statement takes 30 operands, a second one would wait before its own are asked for)
__device__ __forceinline__ uint64_t and_next(const int32_t& a) {
  uint64_t v;
  __builtin_memcpy(&v, &a, 8);
  return v;
}
__device__ __forceinline__ uint32_t workgroup(const SepParams& p, const SepPointwise& q) {
  asm volatile("" ::"s"(q.w), "s"(q.bias), "s"(q.m), "s"(q.s), "s"(q.res), "s"(q.y), "s"(q.relu), "s"(p.ybs), "s"(and_next(p.ypitch)),
               "s"(and_next(p.yragged)), "s"(and_next(p.g_base)), "s"(and_next(p.splits)), "s"(p.per_xcd), "s"(p.splits_inv), "s"(p.tpr_inv),
               "s"(p.x), "s"(p.img), "s"(p.dbias), "s"(p.dm), "s"(p.ds), "s"(p.lut), "s"(p.xbs), "s"(and_next(p.xpitch)), "s"(and_next(p.o16)),
               "s"(and_next(p.units)), "s"(and_next(p.drelu)), "s"(and_next(p.row_lanes_log2)));
  // consecutive workgroups go round-robin to the 8 XCDs: each XCD takes a contiguous run of tiles
  // (neighbours share halo rows, the workgroups of one tile its rows), first of the pair, then of the projection
  return (blockIdx.x & 7) * (uint32_t)p.per_xcd + (blockIdx.x >> 3);
}
__device__ __forceinline__ Place place(const SepParams& p, uint32_t v) {
  Place at;
  const uint32_t tile = __umulhi(v + 1, p.splits_inv);
  at.cs = (int)(v - tile * (uint32_t)p.splits);
  uint32_t above = tile + 1;
  asm("" : "+s"(above));                            // (or the sum is carried out in 64 bits)
  at.b = (int)__umulhi(above, p.tpr_inv);
  const int ti = (int)tile - at.b * p.tpr;
  at.g0 = ti * p.g_base + min(ti, p.g_more);
  at.gn = p.g_base + (ti < p.g_more ? 1 : 0);       // <= MT
  return at;
}
// the first element of batch item b
template <typename T>
__device__ __forceinline__ T* item(T* x, int64_t stride, int b) {
  return x + (uint64_t)(uint32_t)stride * (uint32_t)b;
}

// Toeplitz row m of four taps: bytes 4 - m .. 7 - m of (a weight row's dword, the one before), by one byte permutation
__device__ __forceinline__ uint32_t toeplitz_bytes(int m) { return 0x07060504u - 0x01010101u * (uint32_t)m; }

// Constants of N = 16 or 32 channels in one or two loads per wave: a load of any size holds the address path
// of the unit for 16 cycles, so three 16-channel loads cost as much as 3 KiB of weights.  Lanes [0, N) ask for m,
// [N, 2 N) for s, [2 N, 3 N) for the bias if that fits (N = 16); get() brings a channel's to where it is used.
template <int N>
struct Consts {
  int32_t ms = 0, b = 0;
  bool bias = false;
  __device__ __forceinline__ void load_bias(const int32_t* pb, int c0, int lane) {   // (before the others: it is on one path only)
    bias = pb != nullptr;
    if (N == 32 && pb) b = pb[c0 + (lane & 31)];
  }
  __device__ __forceinline__ void load(const int32_t* pm, const int32_t* ps, const int32_t* pb, int c0, int lane) {
    const int which = lane / N;
    const int32_t* const q = which == 0 ? pm : which == 1 ? ps : (N == 16 && pb) ? pb : pm;
    ms = q[c0 + (lane & (N - 1))];
  }
  // by requests that the caller waits for (N = 32), without a branch between a request and its register's use
  __device__ __forceinline__ void load_by_hand(const int32_t* pm, const int32_t* ps, const int32_t* pb, int c0, int lane) {
    static_assert(N == 32, "m and s in one request");
    bias = pb != nullptr;
    gload4_into(ms, (lane < 32 ? pm : ps) + c0 + (lane & 31));
    gload4_into(b, (bias ? pb : pm) + c0 + (lane & 31));
  }
  __device__ __forceinline__ int32_t get(int32_t v, int from) const { return __builtin_amdgcn_ds_bpermute(4 * from, v); }
  __device__ __forceinline__ int32_t m(int c) const { return get(ms, c); }
  __device__ __forceinline__ int32_t s(int c) const { return get(ms, N + c); }
  __device__ __forceinline__ int32_t bias_of(int c) const { return !bias ? 0 : N == 32 ? get(b, c) : get(ms, 2 * N + c); }
};

__device__ __forceinline__ uint32_t through_table(const unsigned char* lut, uint32_t pk) {
  const uint32_t cd = pk ^ 0x80808080u;
  return (uint32_t)lut[cd & 0xffu] | ((uint32_t)lut[(cd >> 8) & 0xffu] << 8) | ((uint32_t)lut[(cd >> 16) & 0xffu] << 16) |
         ((uint32_t)lut[cd >> 24] << 24);
}

// ---- Tiles of four and seven groups: enough products per step to cover the loads of the next ones.
// (Waves that still have loads to ask for put before those that have not, by s_setprio: without it pairs take 0.998 of the time with it, on
// average over 100 shapes of 256 and 512 channels, 33 to 75 taps, 52 to 51200 frames; single ones over rows of any length 0.97 to 1.02,
// 1.00 on average of 36: nothing, and left out.)
// RAGGED: x or y (and the residual) are the caller's, rows of any length at any address
template <int KCH, int MT, int NA, int NT, bool RAGGED>
__global__ __launch_bounds__(64 * kWaves) void sep_kernel(SepParams p) {
  extern __shared__ __align__(128) unsigned char lds[];   // [Cin][128 B] tile, [kWaves] row buffers and tables
  constexpr int CPW = KCH * 64 / kWaves;            // depthwise channels per wave
  constexpr int NBLK = CPW / 16;                    // in blocks of 16
  constexpr int NL = row_loads(16, MT, NA);
  constexpr bool TIGHT = MT * NT > 8;               // (registers)
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const SepPointwise& pw = p.pw[blockIdx.z];
  const bool proj = blockIdx.z != 0;
  const uint32_t v = workgroup(p, pw);
  if (v >= (uint32_t)p.wgs) return;                 // whole workgroup
  const Place at = place(p, v);
  const int b = at.b, g0 = at.g0, gn = at.gn, cs = at.cs;

  unsigned char* const xs = lds;
  const int rb = row_bytes(p.units, MT, NA) + 256;
  unsigned char* const rows = lds + KCH * 64 * 128 + wave * rb;
  unsigned char* const lut = rows + rb - 256;       // (every wave its own copy: no barrier)
  uint32_t lut_word = 0;
  if (p.lut) lut_word = reinterpret_cast<const uint32_t*>(p.lut)[lane];

  // ---- depthwise half: 16 channels at a time
  const int c_wave = wave * CPW;
  uint32_t xoff[NL];                                // chunk L of 16 rows: chunk L % units of row L / units
#pragma unroll
  for (int j = 0; j < NL; ++j) {
    const int L = lane + 64 * j, ch = (L * p.units_inv) >> 16, c = g0 + p.o16 + L - ch * p.units;
    xoff[j] = (uint32_t)c < (uint32_t)((p.Tin + 15) >> 4) && ch < 16 ? (uint32_t)(ch * p.xpitch + 16 * c) : kNone;
  }
  const int8_t* const xw = item(p.x, p.xbs, b) + (int64_t)c_wave * p.xpitch;
  v4i xr[NL];
  auto tail = [&](int blk) __attribute__((always_inline)) { return blk == NBLK - 1 && wave == kWaves - 1; };
  auto load_rows = [&](int blk) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < NL; ++j) xr[j] = load_chunk<16, RAGGED>(p, xw + (int64_t)(16 * blk) * p.xpitch, tail(blk), xoff[j], 0u);
  };
  auto put_rows = [&](int blk) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      const v4i r = whole_chunk<16, RAGGED>(p, tail(blk), xoff[j], 0u, xr[j]);
      if (lane + 64 * j < 16 * p.units) *reinterpret_cast<v4i*>(rows + 16 * (lane + 64 * j)) = r;
    }
    clear_past_end<16>(p, rows, 16 * p.units, g0 + p.o16, lane);
  };
  const int ch_l = lane >> 2, n_l = lane & 3;
  // weights: rows of 16 NA bytes, each block's over the tile rows that its outputs are written to
  constexpr int NWL = (CPW * NA + 63) / 64;
  static_assert(NA <= 8, "a block's weights fit its tile rows");
  static_assert(16 * (64 * NWL - CPW * NA) <= DwParams::kImageTail, "the last wave's last load ends inside the image");
  unsigned char* const wlds = xs + c_wave * 128;
  const unsigned char* const wrow = wlds + ch_l * (16 * NA);
  const uint32_t sel = toeplitz_bytes(n_l);
  Consts<CPW> dc;
  const unsigned char* const win = rows + ch_l * (16 * p.units) + 4 * (n_l + p.dwoff);
  // dword n_l of group q, row (channel) ch of the tile; the tile's unit q of a row sits in slot q ^ (row & 7)
  const uint32_t tw = (uint32_t)((c_wave + ch_l) * 128 + 4 * n_l) | (uint32_t)((ch_l & 7) << 4);

  // what the pointwise half reads: 16 NT output channels of this wave
  const int n = lane & 15, gi = lane >> 4;
  const int co_w = (cs * kWaves + wave) * 16 * NT;
  v4i wb[3][NT];
  const v4i* const wsrc = reinterpret_cast<const v4i*>(pw.w) + (int64_t)(co_w >> 4) * (KCH * 64) + lane;
  auto load_w = [&](int kc) __attribute__((always_inline)) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) wb[kc % 3][nt] = wsrc[(nt * KCH + kc) * 64];
  };
  Consts<16 * NT> pc;

  if (RAGGED || !proj) {
    dc.load_bias(p.dbias, c_wave, lane);
    v4i wr[NWL];
#pragma unroll
    for (int j = 0; j < NWL; ++j) wr[j] = reinterpret_cast<const v4i*>(p.img)[c_wave * NA + lane + 64 * j];   // (the last wave's into the image's tail)
    load_rows(0);
    dc.load(p.dm, p.ds, p.dbias, c_wave, lane);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < NWL; ++j) {
      const int L = lane + 64 * j;
      if (L < CPW * NA) *reinterpret_cast<v4i*>(wlds + 16 * L + (L < 16 * NA ? 0 : 2048 - 256 * NA)) = wr[j];
    }
    if (p.lut) reinterpret_cast<uint32_t*>(lut)[lane] = lut_word;
#pragma unroll
    for (int blk = 0; blk < NBLK; ++blk) {
      put_rows(blk);
      asm volatile("" ::: "memory");                  // (lanes read what other lanes of the wave wrote: LDS is in order)
      __builtin_amdgcn_sched_barrier(0);
      // window quads a .. a + MT - 1 are what step quad a multiplies; one more is on its way
      uint32_t wd[MT + 1][4], before = 0;
      v4i aq[2];
      auto read_taps = [&](int a) __attribute__((always_inline)) { aq[a & 1] = *reinterpret_cast<const v4i*>(wrow + 2048 * blk + 16 * a); };
      auto read_quad = [&](int a) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) wd[a % (MT + 1)][i] = *reinterpret_cast<const uint32_t*>(win + 16 * a + 4 * i);
      };
      read_taps(0);
#pragma unroll
      for (int a = 0; a < MT; ++a) read_quad(a);
      v4i acc[MT];
      const int32_t db = dc.bias_of(16 * blk + ch_l);
#pragma unroll
      for (int q = 0; q < MT; ++q) acc[q] = (v4i){db, db, db, db};
#pragma unroll
      for (int a = 0; a < NA; ++a) {
        if (a + 1 < NA) {
          read_taps(a + 1);
          read_quad(a + MT);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t d = (uint32_t)aq[a & 1][i], t = __builtin_amdgcn_perm(d, before, sel);
          before = d;
          if (4 * a + i < 4 * (NA - 1) + 1 || 4 * a + i < p.nk) {
#pragma unroll
            for (int q = 0; q < MT; ++q)
              acc[q] = __builtin_amdgcn_mfma_i32_4x4x4i8((int)t, (int)wd[(a + q) % (MT + 1)][i], acc[q], 0, 0, 0);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
        if (a == 1 && blk + 1 < NBLK) load_rows(blk + 1);   // on their way under the rest of the block
      }
      if (blk + 1 == NBLK && !TIGHT) {
        load_w(0);
        load_w(1);
      }
      const int32_t m = dc.m(16 * blk + ch_l), s = dc.s(16 * blk + ch_l);
      auto finish = [&](auto fast_tag, auto relu_tag) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < MT; ++q) {
          const int32_t a4[4] = {acc[q][0], acc[q][1], acc[q][2], acc[q][3]};
          uint32_t pk;
          if constexpr (decltype(fast_tag)::value)
            pk = requant_short4<false, decltype(relu_tag)::value>(a4, m, s - 32, 1 << ((s - 33) & 31), 0u);
          else
            pk = requant_pack4<false, false>(a4, m, s, 0, 0u, p.drelu ? 0 : -128, 127);
          if (p.lut) pk = through_table(lut, pk);
          *reinterpret_cast<uint32_t*>(xs + 16 * 128 * blk + (tw ^ (uint32_t)(q << 4))) = pk;
        }
      };
      if (!__all(s >= kShortMin && s <= kShortMax)) finish(std::false_type{}, std::false_type{});
      else if (p.drelu) finish(std::true_type{}, std::true_type{});
      else finish(std::true_type{}, std::false_type{});
    }
  } else {
    // the projection's tile: unit tid % 8 of rows tid / 8, + 128, ...
    const int u = tid & 7;
    const int8_t* const src = item(p.x, p.xbs, b) + (int64_t)(tid >> 3) * p.xpitch + 16 * (g0 + u);
    v4i r[KCH / 2];
#pragma unroll
    for (int i = 0; i < KCH / 2; ++i)
      if (u < gn) r[i] = *reinterpret_cast<const v4i*>(src + (int64_t)(128 * i) * p.xpitch);
    if (!TIGHT) {
      load_w(0);
      load_w(1);
    }
#pragma unroll
    for (int i = 0; i < KCH / 2; ++i)
      if (u < gn) *reinterpret_cast<v4i*>(xs + ((tid >> 3) + 128 * i) * 128 + ((u ^ (tid >> 3 & 7)) << 4)) = r[i];
  }

  // ---- pointwise half
  if (TIGHT) {
    load_w(0);
    load_w(1);
  }
  pc.load_bias(pw.bias, co_w, lane);
  pc.load(pw.m, pw.s, pw.bias, co_w, lane);
  // residual rows and output rows: lane -> (row lane / 8 of 8, slot lane % 8), the unit in that slot
  const int u_l = (lane & 7) ^ (lane >> 3);
  const bool u_ok = u_l < gn;
  const int t_l = 16 * (g0 + u_l);
  const int64_t yrow = (int64_t)b * p.ybs + (int64_t)(co_w + (lane >> 3)) * p.ypitch;   // of this lane's first row
  v4i rr[NT][2];
  auto load_res = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int8_t* const row = pw.res + yrow + (int64_t)(16 * nt + 8 * h) * p.ypitch;
        if (u_ok) rr[nt][h] = RAGGED && p.yragged ? load_row16(row, t_l, p.Tout) : *reinterpret_cast<const v4i*>(row + t_l);
      }
  };
  __syncthreads();                                  // the tile is complete
  v4i acc[MT][NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int32_t bv = pc.bias_of(16 * nt + n);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt][nt] = (v4i){bv, bv, bv, bv};
  }
  const int l16 = lane & 15, jr = l16 >> 1;
  const uint32_t abase = (uint32_t)((8 * gi + jr) * 128 + 8 * (l16 & 1)) | (uint32_t)(jr << 4);
#pragma unroll
  for (int kc = 0; kc < KCH; ++kc) {
    if (kc + 2 < KCH) load_w(kc + 2);
    if (kc + 2 == KCH && pw.res) load_res();         // (into what the weight ring no longer needs)
    __builtin_amdgcn_sched_barrier(0);
    const unsigned char* ab = xs + kc * 8192;
    v2i ar[3][2];
#pragma unroll
    for (int q = 0; q < 2 && q < MT; ++q) {
      ar[q][0] = read_tr8(ab + (abase ^ (uint32_t)(q << 4)));
      ar[q][1] = read_tr8(ab + (abase ^ (uint32_t)(q << 4)) + 4096);
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const v4i a = {ar[mt % 3][0].x, ar[mt % 3][0].y, ar[mt % 3][1].x, ar[mt % 3][1].y};
      if (mt + 2 < MT) {
        ar[(mt + 2) % 3][0] = read_tr8(ab + (abase ^ (uint32_t)((mt + 2) << 4)));
        ar[(mt + 2) % 3][1] = read_tr8(ab + (abase ^ (uint32_t)((mt + 2) << 4)) + 4096);
      }
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
        acc[mt][nt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, wb[kc % 3][nt], acc[mt][nt], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  int32_t mc[NT], sc[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    mc[nt] = pc.m(16 * nt + n);
    sc[nt] = pc.s(16 * nt + n);
  }

  // ---- epilogue, 16 channels at a time through the wave's own staging block (its row buffer is free):
  // lane (n, gi) holds frames 16 mt + 4 gi + (0..3) of channel 16 nt + n
  const uint32_t sbase = (uint32_t)(n * 128 + 4 * gi) | (uint32_t)((n & 7) << 4);
  bool ok = true;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) ok = ok && sc[nt] >= kShortMin && sc[nt] <= (pw.res ? kShortMaxRes : kShortMax);
  const bool fast = __all(ok);
  const __amdgpu_buffer_rsrc_t yrs = __builtin_amdgcn_make_buffer_rsrc(
      item(pw.y, p.ybs, b) + (int64_t)co_w * p.ypitch, 0, 0x7ffffff0, 0x00027000);
  const uint32_t ylane = (uint32_t)(lane >> 3) * (uint32_t)p.ypitch + (uint32_t)t_l;
  auto epilogue = [&](auto fast_tag, auto res_tag, auto relu_tag) __attribute__((always_inline)) {
    constexpr bool FAST = decltype(fast_tag)::value, RES = decltype(res_tag)::value, RELU = decltype(relu_tag)::value;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      unsigned char* const st = rows;
      if (RES) {
#pragma unroll
        for (int h = 0; h < 2; ++h) *reinterpret_cast<v4i*>(st + 1024 * h + 16 * lane) = rr[nt][h];
        asm volatile("" ::: "memory");
      }
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        uint32_t* const sp = reinterpret_cast<uint32_t*>(st + (sbase ^ (uint32_t)(mt << 4)));
        const int32_t a4[4] = {acc[mt][nt][0], acc[mt][nt][1], acc[mt][nt][2], acc[mt][nt][3]};
        const uint32_t rw = RES ? *sp : 0u;
        if constexpr (FAST)
          *sp = requant_short4<RES, RELU>(a4, mc[nt], sc[nt] - 32, 1 << ((sc[nt] - 33) & 31), rw);
        else
          *sp = requant_pack4<false, true>(a4, mc[nt], sc[nt], 0, rw, pw.relu ? 0 : -128, 127);
        if (mt & 1) __builtin_amdgcn_sched_barrier(0);
      }
      asm volatile("" ::: "memory");
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const v4i o = *reinterpret_cast<const v4i*>(st + 1024 * h + 16 * lane);
        if (RAGGED && p.yragged) {                  // (uniform)
          if (u_ok) store_row16(pw.y + yrow + (int64_t)(16 * nt + 8 * h) * p.ypitch, t_l, p.Tout, o);
          continue;
        }
        const v4u ov = {(unsigned)o.x, (unsigned)o.y, (unsigned)o.z, (unsigned)o.w};
        const uint32_t off = u_ok ? ylane + (uint32_t)(16 * nt + 8 * h) * (uint32_t)p.ypitch : 0xfffffff0u;
        __builtin_amdgcn_raw_buffer_store_b128(ov, yrs, off, 0, kStoreThrough);
      }
    }
  };
  const std::true_type T{};
  const std::false_type F{};
  if (pw.res) {
    if (!fast) epilogue(F, T, F);
    else if (pw.relu) epilogue(T, T, T);
    else epilogue(T, T, F);
  } else {
    if (!fast) epilogue(F, F, F);
    else if (pw.relu) epilogue(T, F, T);
    else epilogue(T, F, F);
  }
}

// The depthwise layer of a wave's CPW channels for MT <= 2 groups of frames: rows and weights by as few requests as can be, weights as
// they are (sep.hip: image), which become Toeplitz rows by one byte permutation per dword.
template <int CPW, int MT, int NA, bool RAGGED>
struct DwSmall {
  static_assert(MT <= 2, "two units per row");
  static constexpr int NL = row_loads(CPW, MT, NA);
  static constexpr int NWL = (CPW * NA + 63) / 64;
  static_assert(16 * (64 * NWL - CPW * NA) <= DwParams::kImageTail, "the last wave's last load ends inside the image");
  Consts<CPW> dc;

  // (the bias first: it is on one path only)
  __device__ __forceinline__ void load_bias(const DwParams& p, int c_wave, int lane) { dc.load_bias(p.dbias, c_wave, lane); }
  // A row's chunks are brought in by 1 << row_lanes_log2 lanes each, so that requests differ by a uniform offset.  (Dividing
  // chunk numbers by the units of a row took 9 vector instructions per request, and each, scalar ones too, is 16 cycles of a unit for 16
  // waves.)  Rows are RU units apart in LDS.
  static constexpr int RU = row_units(MT, NA);
  static constexpr int NX = (CPW << max_row_lanes_log2(MT, NA)) / 64;
  static constexpr int kWeightBytes = NWL * 1024;   // of a wave's weight rows in LDS, NA 16-byte units each
  v4i wr[NWL], xr[NX];
  uint32_t xoff;
  __device__ __forceinline__ uint32_t step(const DwParams& p, int j) const { return (uint32_t)j * (uint32_t)p.row_step; }
  __device__ __forceinline__ void load(const DwParams& p, int b, int g0, int wave, int lane) {
    const int c_wave = wave * CPW;
    // weights: as they lie, whole loads (up to 1008 bytes past a wave's rows: the next wave's, or the image's tail)
    const v4i* const src = reinterpret_cast<const v4i*>(p.img) + c_wave * NA;
#pragma unroll
    for (int j = 0; j < NWL; ++j) wr[j] = src[lane + 64 * j];
    dc.load(p.dm, p.ds, p.dbias, c_wave, lane);
    const int u = lane & ((1 << p.row_lanes_log2) - 1), c = g0 + p.o16 + u;
    xoff = (uint32_t)c < (uint32_t)((p.Tin + 15) >> 4) && u < RU ? (uint32_t)((lane >> p.row_lanes_log2) * p.xpitch + 16 * c) : kNone;
    const int8_t* const xw = item(p.x, p.xbs, b) + (uint64_t)(uint32_t)c_wave * (uint32_t)p.xpitch;
#pragma unroll
    for (int j = 0; j < NX; ++j)                      // (uniform; what is not loaded is not used)
      if (j < 1 || j < CPW >> (6 - p.row_lanes_log2)) xr[j] = load_chunk<CPW, RAGGED>(p, xw, wave == kWaves - 1, xoff, step(p, j));
  }
  // into LDS: CPW rows at rows (small_row_bytes), weight rows at wlds
  __device__ __forceinline__ void lay(const DwParams& p, unsigned char* rows, unsigned char* wlds, int g0, int wave, int lane) {
#pragma unroll
    for (int j = 0; j < NWL; ++j) *reinterpret_cast<v4i*>(wlds + 16 * lane + 1024 * j) = wr[j];
    const int u = lane & ((1 << p.row_lanes_log2) - 1);
    unsigned char* const to = rows + 16 * ((lane >> p.row_lanes_log2) * RU + u);
    if ((1 << max_row_lanes_log2(MT, NA)) <= RU || u < RU) {   // (what lies past a row is the next one's, past the last row the table's)
#pragma unroll
      for (int j = 0; j < NX; ++j)
        if (j < 1 || j < CPW >> (6 - p.row_lanes_log2))
          *reinterpret_cast<v4i*>(to + j * ((1024 * RU) >> p.row_lanes_log2)) =
              whole_chunk<CPW, RAGGED>(p, wave == kWaves - 1, xoff, step(p, j), xr[j]);
    }
    clear_past_end<CPW>(p, rows, 16 * RU, g0 + p.o16, lane);
    asm volatile("" ::: "memory");                    // (lanes read what other lanes of the wave wrote: LDS is in order)
    __builtin_amdgcn_sched_barrier(0);
  }
  // NB blocks of 16 channels from block b0 on, side by side: lane -> channel lane / 4 of the block, frames 4 (lane % 4) + (0..3) of a group
  template <int NB>
  __device__ __forceinline__ void multiply(const DwParams& p, int units, const unsigned char* rows, const unsigned char* wlds, int lane, int b0,
                                           v4i (&dacc)[NB][MT]) const {
    const int ch_l = lane >> 2, n_l = lane & 3;
    const uint32_t sel = toeplitz_bytes(n_l);
    const unsigned char* const win = rows + (16 * b0 + ch_l) * (16 * units) + 4 * (n_l + p.dwoff);
    const unsigned char* const wrow = wlds + (16 * b0 + ch_l) * (16 * NA);
    constexpr int LA = 2, WQ = MT + LA;               // quads read ahead
    uint32_t wd[NB][WQ][4];
    v4i aq[NB][LA + 1];
    uint32_t before[NB];
    auto read_win = [&](int a) __attribute__((always_inline)) {
#pragma unroll
      for (int blk = 0; blk < NB; ++blk)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          wd[blk][a % WQ][i] = *reinterpret_cast<const uint32_t*>(win + 256 * blk * units + 16 * a + 4 * i);
    };
    auto read_taps = [&](int a) __attribute__((always_inline)) {
#pragma unroll
      for (int blk = 0; blk < NB; ++blk) aq[blk][a % (LA + 1)] = *reinterpret_cast<const v4i*>(wrow + 256 * blk * NA + 16 * a);
    };
#pragma unroll
    for (int a = 0; a < LA; ++a) read_taps(a);
#pragma unroll
    for (int a = 0; a < MT + LA - 1; ++a) read_win(a);
#pragma unroll
    for (int blk = 0; blk < NB; ++blk) {
      const int32_t db = dc.bias_of(16 * (b0 + blk) + ch_l);
      before[blk] = 0;
#pragma unroll
      for (int q = 0; q < MT; ++q) dacc[blk][q] = (v4i){db, db, db, db};
    }
#pragma unroll
    for (int a = 0; a < NA; ++a) {
      if (a + LA < NA) {
        read_taps(a + LA);
        read_win(a + MT + LA - 1);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        uint32_t t[NB];
#pragma unroll
        for (int blk = 0; blk < NB; ++blk) {
          const uint32_t d = (uint32_t)aq[blk][a % (LA + 1)][i];
          t[blk] = __builtin_amdgcn_perm(d, before[blk], sel);
          before[blk] = d;
        }
        if (4 * a + i < 4 * (NA - 1) + 1 || 4 * a + i < p.nk) {
#pragma unroll
          for (int q = 0; q < MT; ++q)
#pragma unroll
            for (int blk = 0; blk < NB; ++blk)
              dacc[blk][q] = __builtin_amdgcn_mfma_i32_4x4x4i8((int)t[blk], (int)wd[blk][(a + q) % WQ][i], dacc[blk][q], 0, 0, 0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // put(block, group, the lane's four frames) of the finished blocks
  template <int NB, typename Put>
  __device__ __forceinline__ void finish(const DwParams& p, const unsigned char* lut, int lane, int b0, const v4i (&dacc)[NB][MT], Put put) const {
    const int ch_l = lane >> 2;
#pragma unroll
    for (int blk = 0; blk < NB; ++blk) {
      const int32_t m = dc.m(16 * (b0 + blk) + ch_l), s = dc.s(16 * (b0 + blk) + ch_l);
      auto form = [&](auto fast_tag, auto relu_tag) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < MT; ++q) {
          const int32_t a4[4] = {dacc[blk][q][0], dacc[blk][q][1], dacc[blk][q][2], dacc[blk][q][3]};
          uint32_t pk;
          if constexpr (decltype(fast_tag)::value)
            pk = requant_short4<false, decltype(relu_tag)::value>(a4, m, s - 32, 1 << ((s - 33) & 31), 0u);
          else
            pk = requant_pack4<false, false>(a4, m, s, 0, 0u, p.drelu ? 0 : -128, 127);
          if (p.lut) pk = through_table(lut, pk);
          put(b0 + blk, q, pk);
        }
      };
      if (!__all(s >= kShortMin && s <= kShortMax)) form(std::false_type{}, std::false_type{});
      else if (p.drelu) form(std::true_type{}, std::true_type{});
      else form(std::true_type{}, std::false_type{});
    }
  }
};

// ---- Tiles of one and two groups: launches of few frames, where the products are nothing and the loads
// everything.  A load instruction of any size holds a compute unit's address path for 16 cycles; with 16 waves asking
// for weight images of four bytes per tap, for constants three at a time and for two blocks' rows apart, one workgroup
// (512 -> 256 channels, k = 75) had 592 loads, 9500 of the 15300 cycles it took, and up to ten round trips
// one after the other.  Here
//   - the weights come as they are, zero-padded rows of 16 NA bytes (sep.hip: image), are laid into the
//     wave's own rows of the pointwise tile, which are written later, and become Toeplitz rows by one byte
//     permutation per dword;
//   - rows, weights and constants of all the wave's channels are asked for at once, with them the residual, constants and
//     weights of the pointwise half (of 512 x 32 channels per wave the second half after the depthwise products), and
//     nothing waits in between;
//   - both blocks of 16 channels are multiplied side by side; residual and output rows are two 16-byte
//     units wide, one load and one store per wave.
//   - nothing is merged into a register that is being loaded and no wait stands before the last request (load_chunk), requests
//     differ by uniform offsets, and what every wave would work out for itself is left to the host or done once for all: each
//     instruction, scalar ones above all, is 16 cycles of a unit for 16 waves.  512 -> 512, k = 75 over 50 groups: 13750 -> 12900
//     cycles a workgroup; QuartzNet-5x5, 1 x 1600 frames 180 -> 162 us, 15x5, 1 x 1237 473 -> 424, 32 x 1600 1275 -> 1237, 10x5,
//     8 x 1104 438 -> 404.
// Before the last of these 288 loads, 13400 cycles.  In a chain of such pairs over 50 groups, us a launch: 512 -> 512, k = 75 8.53 -> 7.87,
// 7.54 with KS = 2 below; k = 51 7.91 -> 7.09, 6.67; 256 -> 256, k = 33 5.58 -> 4.99, 4.83.
// KS = 2, where twice as many workgroups still find units of their own: the waves are two groups over the input
// channels of the pointwise half, a workgroup has half as many output channels, its half of the weights and of the
// tile's reads per wave, and the two partial sums meet in LDS.
template <int KCH, int MT, int NA, int NT, int KS, bool RAGGED>
__global__ __launch_bounds__(64 * kWaves) void sep_small_kernel(SepParams p) {
  static_assert(MT <= 2, "two units per staged row");
  extern __shared__ __align__(128) unsigned char lds[];   // [Cin][128 B] tile, [kWaves] row buffers and tables
  constexpr int CPW = KCH * 64 / kWaves;            // depthwise channels per wave
  constexpr int NBLK = CPW / 16;                    // in blocks of 16
  using Dw = DwSmall<CPW, MT, NA, RAGGED>;
  static_assert(Dw::kWeightBytes <= CPW * 128, "weights fit the wave's tile rows");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const SepPointwise& pw = p.pw[blockIdx.z];
  const bool proj = blockIdx.z != 0;
  const uint32_t v = workgroup(p, pw);
  if (v >= (uint32_t)p.wgs) return;                 // whole workgroup
  const Place at = place(p, v);
  const int g0 = at.g0, c_wave = wave * CPW;
  unsigned char* const xs = lds;
  constexpr int rb = small_row_bytes(CPW, row_units(MT, NA), MT, NA) + 256;
  unsigned char* const rows = lds + KCH * 64 * 128 + wave * rb;
  unsigned char* const lut = rows + rb - 256;       // (every wave its own copy: no barrier)
  unsigned char* const wlds = xs + c_wave * 128;
  const int n = lane & 15, gi = lane >> 4;
  constexpr int NWC = kWaves / KS, KC = KCH / KS;   // waves over output channels; chunks per wave
  const int wc = wave % NWC, ks = wave / NWC;
  const int co_w = (at.cs * NWC + wc) * 16 * NT;

  // ---- everything is asked for; what only some launches have comes first, so that the waits for the rest stay exact
  uint32_t lut_word = 0;
  if (p.lut) lut_word = reinterpret_cast<const uint32_t*>(p.lut)[lane];
  Dw dw;
  dw.load_bias(p, c_wave, lane);
  // residual and output: lane -> row lane / 2 of the wave's 16 NT, unit lane % 2
  const int u_l = lane & 1, t_l = 16 * (g0 + u_l);
  const bool y_ok = u_l < at.gn && lane < 32 * NT && ks == 0;
  const int64_t yrow = (int64_t)at.b * p.ybs + (int64_t)(co_w + (lane >> 1)) * p.ypitch;
  v4i rr = {0, 0, 0, 0};
  const uint32_t yoff = y_ok ? (uint32_t)(lane >> 1) * (uint32_t)p.ypitch + (uint32_t)t_l : kNone;
  if (pw.res) {
    if (RAGGED && p.yragged) {
      if (y_ok) rr = load_row16(pw.res + yrow, t_l, p.Tout);
    } else {
      const __amdgpu_buffer_rsrc_t rrs = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<int8_t*>(item(pw.res, p.ybs, at.b)) + (int64_t)co_w * p.ypitch, 0, 0x7ffffff0, 0x00027000);
      rr = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rrs, yoff, 0, 0));
    }
  }
  v4i tr;
  if (RAGGED || !proj) {
    dw.load(p, at.b, g0, wave, lane);
  } else {                                          // the projection's tile: unit tid % 2 of row tid / 2
    const int row0 = 32 * wave;
    const __amdgpu_buffer_rsrc_t xrs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(item(p.x, p.xbs, at.b)) + (int64_t)row0 * p.xpitch, 0,
                                          row0 < 64 * KCH ? 32 * p.xpitch : 0, 0x00027000);
    tr = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(
                                     xrs, u_l < at.gn ? (uint32_t)(lane >> 1) * (uint32_t)p.xpitch + (uint32_t)t_l : kNone, 0, 0));
  }
  // constants of the workgroup's output channels, m | s | bias: 256 of one of them by a wave
  constexpr int CO = NWC * 16 * NT, CL = (CO + 255) / 256;
  int32_t* const cst = reinterpret_cast<int32_t*>(lds + KCH * 64 * 128 + kWaves * rb);
  const int c_of = wave / CL, c_at = 256 * (wave % CL) + 4 * (lane & (CO < 256 ? CO / 4 - 1 : 63));
  v4i cr;
  if (c_of < 3) cr = *reinterpret_cast<const unaligned_chunk16*>((c_of == 0 ? pw.m : c_of == 1 ? pw.s : pw.bias ? pw.bias : pw.m) + at.cs * CO + c_at);
  v4i wb[KC][NT];
  const v4i* const wsrc = reinterpret_cast<const v4i*>(pw.w) + (int64_t)(co_w >> 4) * (KCH * 64) + ks * (KC * 64) + lane;
  auto load_w = [&](int kc) __attribute__((always_inline)) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) wb[kc][nt] = wsrc[(nt * KCH + kc) * 64];
  };
  constexpr int FIRST = KC * NT > 8 ? KC / 2 : KC;  // (registers)
#pragma unroll
  for (int kc = 0; kc < FIRST; ++kc) load_w(kc);
  __builtin_amdgcn_sched_barrier(0);
  if (p.lut) reinterpret_cast<uint32_t*>(lut)[lane] = lut_word;
  auto lay_constants = [&]() __attribute__((always_inline)) {
    if (c_of < 3) *reinterpret_cast<v4i*>(cst + c_of * CO + c_at) = c_of < 2 || pw.bias ? cr : (v4i){0, 0, 0, 0};
  };

  if (RAGGED || !proj) {
    // ---- depthwise half
    dw.lay(p, rows, wlds, g0, wave, lane);
    lay_constants();
    v4i dacc[NBLK][MT];
    dw.template multiply<NBLK>(p, Dw::RU, rows, wlds, lane, 0, dacc);
#pragma unroll
    for (int kc = FIRST; kc < KC; ++kc) load_w(kc);
    // dword n_l of group q, row (channel) ch of the tile; the tile's unit q of a row sits in slot q ^ (row & 7)
    const int ch_l = lane >> 2, n_l = lane & 3;
    const uint32_t tw = (uint32_t)((c_wave + ch_l) * 128 + 4 * n_l) | (uint32_t)((ch_l & 7) << 4);
    dw.template finish<NBLK>(p, lut, lane, 0, dacc, [&](int blk, int q, uint32_t pk) __attribute__((always_inline)) {
      *reinterpret_cast<uint32_t*>(xs + 16 * 128 * blk + (tw ^ (uint32_t)(q << 4))) = pk;
    });
  } else {
    const int row = tid >> 1;
    if (row < 64 * KCH) *reinterpret_cast<v4i*>(xs + row * 128 + ((u_l ^ (row & 7)) << 4)) = tr;
    lay_constants();
#pragma unroll
    for (int kc = FIRST; kc < KC; ++kc) load_w(kc);
  }

  // ---- pointwise half; operand of group mt, chunk kc: item kc MT + mt of one stream, AH of them on their way
  __syncthreads();                                  // the tile is complete
  const int l16 = lane & 15, jr = l16 >> 1;
  const uint32_t abase = (uint32_t)((8 * gi + jr) * 128 + 8 * (l16 & 1)) | (uint32_t)(jr << 4);
  constexpr int AH = 3, AR = AH + 1;
  v2i ar[AR][2];
  auto read_item = [&](int i) __attribute__((always_inline)) {
    const unsigned char* const q = xs + (ks * KC + i / MT) * 8192 + (abase ^ (uint32_t)((i % MT) << 4));
    ar[i % AR][0] = read_tr8(q);
    ar[i % AR][1] = read_tr8(q + 4096);
  };
#pragma unroll
  for (int i = 0; i < AH; ++i) read_item(i);
  v4i acc[MT][NT];
  int32_t mc[NT], sc[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int32_t* const c = cst + 16 * (wc * NT + nt) + n;
    const int32_t bv = ks != 0 ? 0 : c[2 * CO];
    mc[nt] = c[0];
    sc[nt] = c[CO];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt][nt] = (v4i){bv, bv, bv, bv};
  }
#pragma unroll
  for (int i = 0; i < KC * MT; ++i) {
    const v4i a = {ar[i % AR][0].x, ar[i % AR][0].y, ar[i % AR][1].x, ar[i % AR][1].y};
    if (i + AH < KC * MT) read_item(i + AH);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
      acc[i % MT][nt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, wb[i / MT][nt], acc[i % MT][nt], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  }

  if constexpr (KS == 2) {                          // (the row buffers are free)
    static_assert(MT * NT <= 2, "the sums fit a row buffer");
    if (ks == 1) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) *reinterpret_cast<v4i*>(rows + 1024 * (mt * NT + nt) + 16 * lane) = acc[mt][nt];
    }
    __syncthreads();
    if (ks == 1) return;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc[mt][nt] += *reinterpret_cast<const v4i*>(rows + NWC * rb + 1024 * (mt * NT + nt) + 16 * lane);
  }

  // ---- epilogue through the wave's own staging block (its row buffer is free), 32 bytes per channel: lane
  // (n, gi) holds frames 16 mt + 4 gi + (0..3) of channel 16 nt + n
  unsigned char* const st = rows;
  bool ok = true;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) ok = ok && sc[nt] >= kShortMin && sc[nt] <= (pw.res ? kShortMaxRes : kShortMax);
  const bool fast = __all(ok);
  auto epilogue = [&](auto fast_tag, auto res_tag, auto relu_tag) __attribute__((always_inline)) {
    constexpr bool FAST = decltype(fast_tag)::value, RES = decltype(res_tag)::value, RELU = decltype(relu_tag)::value;
    if (RES) {
      if (lane < 32 * NT) *reinterpret_cast<v4i*>(st + 16 * lane) = rr;
      asm volatile("" ::: "memory");
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        uint32_t* const sp = reinterpret_cast<uint32_t*>(st + 32 * (16 * nt + n) + 16 * mt + 4 * gi);
        const int32_t a4[4] = {acc[mt][nt][0], acc[mt][nt][1], acc[mt][nt][2], acc[mt][nt][3]};
        const uint32_t rw = RES ? *sp : 0u;
        if constexpr (FAST)
          *sp = requant_short4<RES, RELU>(a4, mc[nt], sc[nt] - 32, 1 << ((sc[nt] - 33) & 31), rw);
        else
          *sp = requant_pack4<false, true>(a4, mc[nt], sc[nt], 0, rw, pw.relu ? 0 : -128, 127);
      }
    asm volatile("" ::: "memory");
  };
  const std::true_type T{};
  const std::false_type F{};
  if (pw.res) {
    if (!fast) epilogue(F, T, F);
    else if (pw.relu) epilogue(T, T, T);
    else epilogue(T, T, F);
  } else {
    if (!fast) epilogue(F, F, F);
    else if (pw.relu) epilogue(T, F, T);
    else epilogue(T, F, F);
  }
  const v4i o = *reinterpret_cast<const v4i*>(st + 16 * (lane & (32 * NT - 1)));
  if (RAGGED && p.yragged) {                        // (uniform)
    if (y_ok) store_row16(pw.y + yrow, t_l, p.Tout, o);
  } else {
    const __amdgpu_buffer_rsrc_t yrs = __builtin_amdgcn_make_buffer_rsrc(
        item(pw.y, p.ybs, at.b) + (int64_t)co_w * p.ypitch, 0, 0x7ffffff0, 0x00027000);
    const v4u ov = {(unsigned)o.x, (unsigned)o.y, (unsigned)o.z, (unsigned)o.w};
    __builtin_amdgcn_raw_buffer_store_b128(ov, yrs, yoff, 0, kStoreThrough);
  }
}

template <int KCH, int MT, int NA, int NT, int KS, bool RAGGED>
hipError_t launch_t(const SepParams& p, size_t lds, hipStream_t st) {
  static std::atomic<uint64_t> lds_raised{0};   // per instantiation, a bit per device
  void (*kernel)(SepParams);
  if constexpr (MT <= 2) kernel = sep_small_kernel<KCH, MT, NA, NT, KS, RAGGED>;
  else kernel = sep_kernel<KCH, MT, NA, NT, RAGGED>;
  if (const hipError_t e = ensure_max_dynamic_lds((const void*)kernel, lds_raised); e != hipSuccess) return e;
  return launch_kernel(kernel, dim3((unsigned)(8 * p.per_xcd), 1, p.pw[1].w ? 2 : 1), dim3(64 * kWaves), lds, st, p);
}

// the instantiations of one tap range (ragged rows: at most 4 groups, more do not fit the registers)
template <int NA>
hipError_t launch_na(const SepChoice& c, const SepParams& p, size_t lds, hipStream_t st) {
#define QASR_CASE(K, M, N, S, R) if (c.KCH == K && c.MT == M && c.NT == N && c.KS == S && c.ragged == R) return launch_t<K, M, NA, N, S, R>(p, lds, st);
#define QASR_MTS(K, N) QASR_CASE(K, 1, N, 1, false) QASR_CASE(K, 2, N, 1, false) QASR_CASE(K, 4, N, 1, false) QASR_CASE(K, 7, N, 1, false) \
                       QASR_CASE(K, 1, N, 1, true) QASR_CASE(K, 2, N, 1, true) QASR_CASE(K, 4, N, 1, true)
  QASR_MTS(4, 1) QASR_MTS(4, 2) QASR_MTS(8, 1) QASR_MTS(8, 2)
  QASR_CASE(4, 1, 1, 2, false) QASR_CASE(4, 2, 1, 2, false) QASR_CASE(8, 1, 1, 2, false) QASR_CASE(8, 2, 1, 2, false)
  QASR_CASE(4, 1, 1, 2, true) QASR_CASE(4, 2, 1, 2, true) QASR_CASE(8, 1, 1, 2, true) QASR_CASE(8, 2, 1, 2, true)
#undef QASR_MTS
#undef QASR_CASE
  return hipErrorInvalidValue;
}

}  // namespace sep
}  // namespace qasr
