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
// dw_pipe.hip the operand is 4 instead of 16 bytes per tap, small enough to be read as a prebuilt image,
// and a tile of a few groups wastes no columns (16 x 16 x 64 wants 256 frames of a channel).  It runs
// at 10 cycles per product, (k + 3) / 4 products per 16 frames of 16 channels: at k = 75 that is 5 us
// for 512 channels x 112 frames.  The window dwords are read one by one: a 16-byte LDS read at a 4-byte aligned
// address measured 59 cycles against 16.
//
// Pointwise half: as pw_pipe_body.hpp (transposing LDS reads, packed weights straight from L2), one
// pass of 16 NT channels per wave, compiler-visible loads.
#pragma once
#include "sep.hpp"

#include <type_traits>

namespace qasr {
namespace sep {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));

constexpr int kStoreThrough = 17;    // sc0 sc1: the output rows are written through (see pw_pipe_body.hpp)
constexpr int kWaves = 16;           // 4 per SIMD: each phase's latencies pass under another wave's products
constexpr int kMaxUnits = 15;        // chunks per row in LDS: 16 rows are at most four 64-lane loads

__device__ __forceinline__ v2i read_tr8(const unsigned char* p) {
  return __builtin_amdgcn_ds_read_tr8_b64_v2i32(
      (v2i __attribute__((address_space(3)))*)(const_cast<unsigned char*>(p)));
}

// bytes of a wave's row buffer: 16 rows and what the windows of the last row read past it, at least
// the 16 x 128 bytes of the output staging
__host__ __device__ inline int row_bytes(int units, int MT, int NA) {
  const int rows = 15 * 16 * units + 16 * (MT + NA) + 32;
  return ((rows > 2048 ? rows : 2048) + 15) & ~15;
}

// RAGGED: x or y (and the residual) are the caller's, rows of any length at any address
template <int KCH, int MT, int NA, int NT, bool RAGGED>
__global__ __launch_bounds__(64 * kWaves) void sep_kernel(SepParams p) {
  extern __shared__ __align__(128) unsigned char lds[];   // [Cin][128 B] tile, [kWaves] row buffers, table
  constexpr int CPW = KCH * 64 / kWaves;            // depthwise channels per wave
  constexpr int NBLK = CPW / 16;                    // in blocks of 16
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // consecutive workgroups go round-robin to the 8 XCDs: each XCD takes a contiguous run of tiles
  // (neighbours share halo rows, the workgroups of one tile its rows)
  const int v = (int)(blockIdx.x & 7) * p.per_xcd + (int)(blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= p.per_xcd || v >= p.wgs) return;                 // whole workgroup
  const int tile = v / p.splits, cs = v - tile * p.splits;
  const int b = tile / p.tpr, ti = tile - b * p.tpr;
  const int g0 = (int)((int64_t)ti * p.gpr / p.tpr), gn = (int)((int64_t)(ti + 1) * p.gpr / p.tpr) - g0;   // gn <= MT

  unsigned char* const xs = lds;
  const int rb = row_bytes(p.units, MT, NA);
  unsigned char* const rows = lds + KCH * 64 * 128 + wave * rb;
  unsigned char* const lut = lds + KCH * 64 * 128 + kWaves * rb;
  if (p.lut && tid < 64) reinterpret_cast<uint32_t*>(lut)[tid] = reinterpret_cast<const uint32_t*>(p.lut)[tid];

  // ---- depthwise half: 16 channels at a time.  Chunk L of the 16 rows (row L / units, chunk L % units)
  // is loaded by lane L % 64; chunks outside [0, Tin) are zero, the chunk a row ends in is masked.
  const int c_wave = wave * CPW;
  int32_t xoff[4];                                  // byte offset of the chunk within the 16 rows
  uint32_t in = 0, last = 0;                        // bit j: chunk j has frames; ... and its row ends inside it
  const int t_last = p.Tin & ~15;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int L = lane + 64 * j, ch = L / p.units, u = L - ch * p.units;
    const int t = 16 * (g0 + p.o16 + u);
    if (ch < 16 && t >= 0 && t < p.Tin) in |= 1u << j;
    if (t == t_last) last |= 1u << j;
    xoff[j] = ch * p.xpitch + t;
  }
  const int8_t* const xw = p.x + (int64_t)b * p.xbs + (int64_t)c_wave * p.xpitch;
  v4i xr[4];
  auto load_rows = [&](int blk) __attribute__((always_inline)) {
    const int8_t* const src = xw + (int64_t)(16 * blk) * p.xpitch;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      xr[j] = (v4i){0, 0, 0, 0};
      if (in & (1u << j)) {
        if (RAGGED && (last & (1u << j))) xr[j] = load_row16(src + xoff[j] - t_last, t_last, p.Tin);
        else xr[j] = *reinterpret_cast<const unaligned_chunk16*>(src + xoff[j]);
      }
    }
  };
  auto put_rows = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (!RAGGED && (last & (1u << j))) xr[j] = keep_bytes(xr[j], p.Tin & 15);
      if (lane + 64 * j < 16 * p.units) *reinterpret_cast<v4i*>(rows + 16 * (lane + 64 * j)) = xr[j];
    }
  };
  const int ch_l = lane >> 2, n_l = lane & 3;
  v4i aw[3];                                        // weight quads, two steps ahead
  int32_t db, dm, dsv;
  const v4i* const asrc = reinterpret_cast<const v4i*>(p.img) + (int64_t)(wave * NBLK) * (NA * 64) + lane;
  auto load_quad_weights = [&](int blk, int a) __attribute__((always_inline)) { aw[a % 3] = asrc[(blk * NA + a) * 64]; };
  auto load_weights = [&](int blk) __attribute__((always_inline)) {
    load_quad_weights(blk, 0);
    load_quad_weights(blk, 1);
    const int c = c_wave + 16 * blk + ch_l;
    db = p.dbias ? p.dbias[c] : 0;
    dm = p.dm[c];
    dsv = p.ds[c];
  };
  const unsigned char* const win = rows + ch_l * (16 * p.units) + 4 * (n_l + p.dwoff);
  // dword n_l of group q, row (channel) ch of the tile; the tile's unit q of a row sits in slot q ^ (row & 7)
  const uint32_t tw = (uint32_t)((c_wave + ch_l) * 128 + 4 * n_l) | (uint32_t)((ch_l & 7) << 4);

  load_rows(0);
  load_weights(0);
  if (p.lut) __syncthreads();                       // (the table is complete)
#pragma unroll
  for (int blk = 0; blk < NBLK; ++blk) {
    put_rows();
    asm volatile("" ::: "memory");                  // (lanes read what other lanes of the wave wrote: LDS is in order)
    __builtin_amdgcn_sched_barrier(0);
    // window quads a .. a + MT - 1 are what step quad a multiplies; one more is on its way
    uint32_t wd[MT + 1][4];
    auto read_quad = [&](int a) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < 4; ++i) wd[a % (MT + 1)][i] = *reinterpret_cast<const uint32_t*>(win + 16 * a + 4 * i);
    };
#pragma unroll
    for (int a = 0; a < MT; ++a) read_quad(a);
    v4i acc[MT];
#pragma unroll
    for (int q = 0; q < MT; ++q) acc[q] = (v4i){db, db, db, db};
#pragma unroll
    for (int a = 0; a < NA; ++a) {
      if (a + 1 < NA) read_quad(a + MT);
      if (a + 2 < NA) load_quad_weights(blk, a + 2);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (4 * a + i < 4 * (NA - 1) + 1 || 4 * a + i < p.nk) {
#pragma unroll
          for (int q = 0; q < MT; ++q)
            acc[q] = __builtin_amdgcn_mfma_i32_4x4x4i8(aw[a % 3][i], (int)wd[(a + q) % (MT + 1)][i], acc[q], 0, 0, 0);
        }
      __builtin_amdgcn_sched_barrier(0);
      if (a == 1 && blk + 1 < NBLK) load_rows(blk + 1);   // on their way under the rest of the block
    }
    const int32_t m = dm, s = dsv;
    if (blk + 1 < NBLK) load_weights(blk + 1);
    auto finish = [&](auto fast_tag, auto relu_tag) __attribute__((always_inline)) {
#pragma unroll
      for (int q = 0; q < MT; ++q) {
        const int32_t a4[4] = {acc[q][0], acc[q][1], acc[q][2], acc[q][3]};
        uint32_t pk;
        if constexpr (decltype(fast_tag)::value)
          pk = requant_short4<false, decltype(relu_tag)::value>(a4, m, s - 32, 1 << ((s - 33) & 31), 0u);
        else
          pk = requant_pack4<false, false>(a4, m, s, 0, 0u, p.drelu ? 0 : -128, 127);
        if (p.lut) {
          const uint32_t cd = pk ^ 0x80808080u;
          pk = (uint32_t)lut[cd & 0xffu] | ((uint32_t)lut[(cd >> 8) & 0xffu] << 8) |
               ((uint32_t)lut[(cd >> 16) & 0xffu] << 16) | ((uint32_t)lut[cd >> 24] << 24);
        }
        *reinterpret_cast<uint32_t*>(xs + 16 * 128 * blk + (tw ^ (uint32_t)(q << 4))) = pk;
      }
    };
    if (!__all(s >= kShortMin && s <= kShortMax)) finish(std::false_type{}, std::false_type{});
    else if (p.drelu) finish(std::true_type{}, std::true_type{});
    else finish(std::true_type{}, std::false_type{});
  }

  // ---- pointwise half: 16 NT output channels of this wave
  const int n = lane & 15, gi = lane >> 4;
  const int co_w = (cs * kWaves + wave) * 16 * NT;
  v4i wb[3][NT];
  const v4i* const wsrc = reinterpret_cast<const v4i*>(p.w) + (int64_t)(co_w >> 4) * (KCH * 64) + lane;
  auto load_w = [&](int kc, v4i (&dst)[NT]) __attribute__((always_inline)) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) dst[nt] = wsrc[(nt * KCH + kc) * 64];
  };
  load_w(0, wb[0]);
  load_w(1, wb[1]);
  int32_t mc[NT], sc[NT];
  v4i acc[MT][NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int co = co_w + 16 * nt + n;
    const int32_t bv = p.bias ? p.bias[co] : 0;
    mc[nt] = p.m[co];
    sc[nt] = p.s[co];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt][nt] = (v4i){bv, bv, bv, bv};
  }
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
        const int8_t* const row = p.res + yrow + (int64_t)(16 * nt + 8 * h) * p.ypitch;
        if (u_ok) rr[nt][h] = RAGGED && p.yragged ? load_row16(row, t_l, p.Tout) : *reinterpret_cast<const v4i*>(row + t_l);
      }
  };
  __syncthreads();                                  // the tile is complete
  const int l16 = lane & 15, jr = l16 >> 1;
  const uint32_t abase = (uint32_t)((8 * gi + jr) * 128 + 8 * (l16 & 1)) | (uint32_t)(jr << 4);
#pragma unroll
  for (int kc = 0; kc < KCH; ++kc) {
    if (kc + 2 < KCH) load_w(kc + 2, wb[(kc + 2) % 3]);
    if (kc + 2 == KCH && p.res) load_res();         // (into what the weight ring no longer needs)
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

  // ---- epilogue, 16 channels at a time through the wave's own staging block (its row buffer is free):
  // lane (n, gi) holds frames 16 mt + 4 gi + (0..3) of channel 16 nt + n
  const uint32_t sbase = (uint32_t)(n * 128 + 4 * gi) | (uint32_t)((n & 7) << 4);
  bool ok = true;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) ok = ok && sc[nt] >= kShortMin && sc[nt] <= (p.res ? kShortMaxRes : kShortMax);
  const bool fast = __all(ok);
  const __amdgpu_buffer_rsrc_t yrs = __builtin_amdgcn_make_buffer_rsrc(
      p.y + (int64_t)b * p.ybs + (int64_t)co_w * p.ypitch, 0, 0x7ffffff0, 0x00027000);
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
          *sp = requant_pack4<false, true>(a4, mc[nt], sc[nt], 0, rw, p.relu ? 0 : -128, 127);
        if (mt & 1) __builtin_amdgcn_sched_barrier(0);
      }
      asm volatile("" ::: "memory");
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const v4i o = *reinterpret_cast<const v4i*>(st + 1024 * h + 16 * lane);
        if (RAGGED && p.yragged) {                  // (uniform)
          if (u_ok) store_row16(p.y + yrow + (int64_t)(16 * nt + 8 * h) * p.ypitch, t_l, p.Tout, o);
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
  if (p.res) {
    if (!fast) epilogue(F, T, F);
    else if (p.relu) epilogue(T, T, T);
    else epilogue(T, T, F);
  } else {
    if (!fast) epilogue(F, F, F);
    else if (p.relu) epilogue(T, F, T);
    else epilogue(T, F, F);
  }
}

template <int KCH, int MT, int NA, int NT, bool RAGGED>
hipError_t launch_t(const SepParams& p, size_t lds, hipStream_t st) {
  static std::atomic<uint64_t> lds_raised{0};   // per instantiation, a bit per device
  if (const hipError_t e = ensure_max_dynamic_lds((const void*)sep_kernel<KCH, MT, NA, NT, RAGGED>, lds_raised); e != hipSuccess)
    return e;
  return launch_kernel(sep_kernel<KCH, MT, NA, NT, RAGGED>, dim3((unsigned)(8 * p.per_xcd)), dim3(64 * kWaves), lds, st, p);
}

// the instantiations of one tap range (ragged rows: at most 4 groups, more do not fit the registers)
template <int NA>
hipError_t launch_na(const SepChoice& c, const SepParams& p, size_t lds, hipStream_t st) {
#define QASR_CASE(K, M, N, R) if (c.KCH == K && c.MT == M && c.NT == N && c.ragged == R) return launch_t<K, M, NA, N, R>(p, lds, st);
#define QASR_MTS(K, N) QASR_CASE(K, 1, N, false) QASR_CASE(K, 2, N, false) QASR_CASE(K, 4, N, false) QASR_CASE(K, 7, N, false) \
                       QASR_CASE(K, 1, N, true) QASR_CASE(K, 2, N, true) QASR_CASE(K, 4, N, true)
  QASR_MTS(4, 1) QASR_MTS(4, 2) QASR_MTS(8, 1) QASR_MTS(8, 2)
#undef QASR_MTS
#undef QASR_CASE
  return hipErrorInvalidValue;
}

}  // namespace sep
}  // namespace qasr
