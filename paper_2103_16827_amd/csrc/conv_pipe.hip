// Dense int8 convolution (k >= 2 taps, any stride / dilation) as an implicit GEMM on the gfx950
// int8 matrix cores (v_mfma_i32_16x16x64_i8), software-pipelined over the contraction, with the
// fused epilogue (bias, dyadic rescale, residual, clamp).
//
//     Y[t, co] = sum_j sum_ci X[ci, t*stride - pad_left + j*dilation] * W[j][co][ci]
//
// Roles and layouts are those of gemm_mfma.hip: the A operand is the activation tile transposed
// (rows = output frames, K = input channels), the B operand the weight tile (packed form: 1 KiB
// contiguous per wave-wide load); a workgroup owns 16 MT output frames of one batch item and 64 NT
// output channels, 16 NT for each of the 4 waves of a group (up to four groups share the taps); each 64-channel chunk of the tile (with the time
// halo the taps need) is transposed in registers (4x4 byte blocks, v_perm_b32) into LDS rows
// [frame][64 channels], 80-byte pitch, so that a tap is a row offset.
//
// What differs is the order in time.  gemm_mfma loads and transposes a chunk, synchronises,
// multiplies its k taps, synchronises: the memory latency of every chunk and the L2 latency of
// every tap's weights are exposed.  Here the contraction is one flat stream of (chunk, tap) steps:
//   - the weights of step q + 3 are requested while step q is multiplied (ring of four);
//   - the global loads of chunk c + 2 are issued in the middle of chunk c, right after chunk c + 1 has been
//     transposed into LDS (three LDS buffers, one barrier per chunk, in its middle), so that the operand
//     reads run ahead across chunks too.
// All these requests are counted by hand (vmem.hpp).  Where the compiler counted them, it had to join the paths
// with and without a chunk on its way: two steps of three waited for weights asked for one step
// earlier, the step after a chunk's request for the whole chunk, and every step for its last operand reads (16 x 800
// frames, ring of three: 768 channels, 25 taps 150 -> 142 us, 512 channels, 17 taps 62 -> 58, 256, 11 taps 22 -> 17).
// What bounds the rest: on operands that are not zeros the chip does not hold its clock.  A plain loop of such
// products (compiler's waits, 80 x 64 per wave), on random codes / on zeros: from registers 4.0 / 4.9 POP/s, with the
// activations from LDS 3.6 / 4.4, with the weights from the L2 as well 2.7 / 3.9; 160 x 32 per wave 4.15 / 5.0, 3.1 / 3.8,
// 2.8 / 3.7.  The 768-channel layers of 16 x 800 frames run at 2.59, in 480 tiles of at most 512 at once.
// Small layers are bound by the number of workgroups instead: the tile (16 MT frames x 64 NT channels), the groups that
// share its taps and the workgroups that share its chunks are chosen per layer by a model of cycles (unit_cycles).
#include "kernels.hpp"
#include "tuning.hpp"
#include "vmem.hpp"

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <type_traits>

namespace qasr {

namespace {

typedef unsigned v4u __attribute__((ext_vector_type(4)));

constexpr int kStoreThrough = 17;   // sc0 sc1: partial sums are written through, which leaves the release little to write back
constexpr int kMaxSplits = 8;

constexpr int kXS = 80;       // LDS row pitch in bytes: 64 channels + 16 pad
constexpr int kConstBytes = 4 * 768;   // per wave of a group: m, s and bias of up to 64 channels
constexpr int kW = 4;         // weight ring: the step multiplied and three on their way
constexpr int kMaxRows = 256; // one 4-frame x 16-channel unit per thread and chunk

struct CpGeom {
  int n_tt, n_co;     // frame tiles per batch item, channel tiles
  int rows;           // LDS rows (input frames incl. halo, rounded to 4)
  int kchunks;        // Cin / 64
  int co16n;          // ceil(Cout / 16)
  int splits;         // workgroups per tile, each with a range of the chunks
  int tiles;          // B * n_tt * n_co * splits
  int per_xcd;        // ceil(tiles / 8): tiles of one XCD (the grid is 8 * per_xcd workgroups)
  float r_nbt, r_splits, r_tt;   // reciprocals of B * n_tt, splits, n_tt
  int fq_inv;         // ceil(2^16 / (rows / 4)): x / (rows / 4) = x fq_inv >> 16 for x < 256, rows <= 256
};

// KG > 1: the taps of a chunk are split over KG groups of 4 waves that share the chunk in LDS, and their
// accumulators are summed through LDS at the end.  A launch with fewer tiles than the chip has SIMDs to
// feed leaves one wave per SIMD, which spends most of a step waiting (a 64 x 128 tile: 128 cycles of
// products, 380 per step); with four groups the latencies pass under the other groups' products.
template <int MT, int NT, int KG>
__global__ __launch_bounds__(256 * KG) void conv_pipe_kernel(ConvParams p, CpGeom g) {
  extern __shared__ __align__(16) unsigned char xs[];   // [3 buffers][rows][kXS]; KG > 1: the partial sums after that
  constexpr int TM = 16 * MT, TN = 64 * NT;
  // All arguments of the loop in one go, and no integer division in front of the first load: with 16 waves the
  // seven divisions and a dozen dependent scalar loads took 6900 cycles of the 25800 of a 256-channel layer of 800 frames.
  // (Those of the epilogue only where they need no spill: not in the tall tiles of two groups.  n_co is asked for and not
  // used: without it the registers fall otherwise and 16 x 1600 frames of a Jasper take 3671 us for 3652.)
  asm volatile("" ::"s"(p.x), "s"(p.w), "s"(p.xbs), "s"(p.B), "s"(p.Tin), "s"(p.k), "s"(p.stride), "s"(p.dil), "s"(p.pl), "s"(p.xpad));
  if constexpr (KG == 1 || MT < 8) asm volatile("" ::"s"(p.bias), "s"(p.m), "s"(p.s), "s"(p.Cout));
  asm volatile("" ::"s"(g.n_tt), "s"(g.n_co), "s"(g.rows), "s"(g.kchunks), "s"(g.co16n), "s"(g.splits), "s"(g.tiles), "s"(g.per_xcd),
               "s"(g.r_nbt), "s"(g.r_splits), "s"(g.r_tt), "s"(g.fq_inv));

  const int tid = threadIdx.x & 255, lane = tid & 63, wave = tid >> 6;   // within the group
  const int kg = KG > 1 ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 8)) : 0;
  const int j0 = KG > 1 ? kg * p.k / KG : 0, j1 = KG > 1 ? (kg + 1) * p.k / KG : p.k;   // this group's taps
  const int n = lane & 15, gi = lane >> 4;

  // Workgroup -> tile.  Consecutive workgroups go round-robin to the 8 XCDs, each with an L2 of its
  // own, and every workgroup streams the whole weight slice of its channel tile: so the tiles are
  // numbered channel tile first (slowest), then batch item, then frame tile, and XCD x takes the
  // contiguous run [x per_xcd, (x + 1) per_xcd) of that order.  An XCD then touches one channel tile,
  // two where its run crosses a boundary, instead of all of them, and its workgroups, which start
  // together and step through the same (chunk, tap) sequence, share each weight line while it is
  // in that L2; neighbouring frame tiles (shared halo lines) stay on one XCD as well.
  // (per_xcd == 0, a tuning override: the plain order, tile = workgroup index, for comparisons)
  const int v = g.per_xcd ? (int)(blockIdx.x & 7) * g.per_xcd + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
  if (v >= g.tiles) return;                         // whole workgroup, before any barrier
  const int nbt = p.B * g.n_tt;
  const int cs = divide_uniform(v, nbt, g.r_nbt), bt = v - cs * nbt;   // bt: (b, t_tile) of the tile
  const int co_tile = g.splits == 1 ? cs : divide_uniform(cs, g.splits, g.r_splits), split = cs - co_tile * g.splits;
  int c0 = 0, nkc = g.kchunks;                      // this workgroup's chunks
  if (g.splits > 1) {
    c0 = divide_uniform(split * g.kchunks, g.splits, g.r_splits);
    nkc = divide_uniform((split + 1) * g.kchunks, g.splits, g.r_splits) - c0;
  }
  const int b = divide_uniform(bt, g.n_tt, g.r_tt), t_tile = bt - b * g.n_tt;

  const int t0 = t_tile * TM;                       // first output frame of the tile
  const int f0 = t0 * p.stride - p.pl;              // first input frame the tile reads
  const int fa = f0 & ~3;                           // rounded down to a dword (also if negative)
  const int foff = f0 - fa;
  const int co_w = co_tile * TN + wave * 16 * NT;   // first output channel of this wave
  const int bufbytes = g.rows * kXS;

  const int8_t* xb = p.x + (int64_t)b * p.xbs + (int64_t)(64 * c0) * (p.Tin + p.xpad);

  // ---- activation chunk kc: global -> registers (issue), registers -> LDS transposed (commit).
  // A thread owns one unit of the chunk: frames 4 fq..+4 of the 16 channels that make one 16-byte
  // column group cg of the LDS rows (four 4x4 byte blocks, channel quads 2cg, 2cg+1, 2cg+8,
  // 2cg+9 in the operand order).  It writes four 16-byte rows; lanes with consecutive fq are
  // 320 bytes apart, which is 16 banks, so the four rows are written in an order rotated by
  // (fq >> 2) & 3: then 16 consecutive lanes cover all 64 banks.  The rotation costs nothing: it
  // is folded into the byte selectors of the first transposition stage.
  const int nfq = g.rows >> 2;                      // frame quads per chunk (<= 64)
  const int u_cg = (tid * g.fq_inv) >> 16, u_fq = tid - u_cg * nfq;
  const int rot = (u_fq >> 2) & 3;
  const int u_f = fa + 4 * u_fq;                    // first input frame of the unit
  const bool u_on = u_cg < 4 && u_f >= 0 && u_f < p.Tin;
  const int xpitch = p.Tin + p.xpad;
  // A unit at a row's end whose last frames do not exist is loaded from inside the row (any byte
  // address will do) and shifted down: the missing frames come out as the implicit zeros.
  const int u_fl = min(u_f, p.Tin - 4);
  const int u_shr = u_on ? 8 * (u_f - u_fl) : 0;
  const uint32_t xoff = u_on ? (uint32_t)(8 * u_cg * xpitch + u_fl) : 0u;   // (Cin x pitch < 2^31)
  uint32_t sel_lo, sel_hi;                          // frames rot, rot+1 | rot+2, rot+3 of two rows
  {
    const uint32_t f0s = rot, f1s = (rot + 1) & 3, f2s = (rot + 2) & 3, f3s = (rot + 3) & 3;
    sel_lo = f0s | ((4 + f0s) << 8) | (f1s << 16) | ((4 + f1s) << 24);
    sel_hi = f2s | ((4 + f2s) << 8) | (f3s << 16) | ((4 + f3s) << 24);
  }
  // (every wave asks for all 16 dwords, whichever of its lanes take part: the waits below count requests)
  int32_t xr[4][4];
  auto issue_chunk = [&](int kc) __attribute__((always_inline)) {
    const int8_t* base = xb + (int64_t)(64 * kc) * xpitch;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int c = 4 * ((i & 1) + 8 * (i >> 1)) + e;
        xr[i][e] = gload4(base + (int64_t)c * xpitch, xoff);
      }
  };
  auto commit_chunk = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) tie(xr[i][e]);
    if (u_cg < 4) {
      unsigned char* dst = xs + buf * bufbytes + 4 * u_fq * kXS + 16 * u_cg;
      uint32_t c[4][4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        uint32_t r[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = u_on ? (uint32_t)xr[i][e] >> u_shr : 0u;
        // r_e = 4 consecutive frames of channel e  ->  c_e = 4 consecutive channels of frame
        // (e + rot) & 3
        const uint32_t lo01 = __builtin_amdgcn_perm(r[1], r[0], sel_lo);
        const uint32_t hi01 = __builtin_amdgcn_perm(r[1], r[0], sel_hi);
        const uint32_t lo23 = __builtin_amdgcn_perm(r[3], r[2], sel_lo);
        const uint32_t hi23 = __builtin_amdgcn_perm(r[3], r[2], sel_hi);
        c[i][0] = __builtin_amdgcn_perm(lo23, lo01, 0x05040100u);
        c[i][1] = __builtin_amdgcn_perm(lo23, lo01, 0x07060302u);
        c[i][2] = __builtin_amdgcn_perm(hi23, hi01, 0x05040100u);
        c[i][3] = __builtin_amdgcn_perm(hi23, hi01, 0x07060302u);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
        *reinterpret_cast<v4i*>(dst + ((e + rot) & 3) * kXS) =
            (v4i){(int)c[0][e], (int)c[1][e], (int)c[2][e], (int)c[3][e]};
    }
  };

  // ---- weights: step q = (chunk, tap) of the flat contraction, ring of kW steps
  const int Q = nkc * (j1 - j0);
  int wkc = 0, wj = j0;                             // chunk and tap of the next step to request
  // (the packed buffer is below 2 GiB: a wave-uniform base per step plus a 32-bit lane offset)
  uint32_t woff[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
    woff[nt] = (uint32_t)((min((co_w >> 4) + nt, g.co16n - 1) * g.kchunks * 64 + lane) * 16);
  v4i wb[kW][NT];
  auto load_w = [&](int nt, v4i (&dst)[NT]) __attribute__((always_inline)) {
    dst[nt] = gload16(p.w + (int64_t)(wj * g.co16n * g.kchunks + c0 + wkc) * 1024, woff[nt]);
  };
  auto next_w = [&]() __attribute__((always_inline)) {
    if (++wj == j1) {                               // (the stream stays on its last step at the end)
      if (wkc + 1 < nkc) { wj = j0; ++wkc; } else { --wj; }
    }
  };

  // ---- prologue: constants (output channels clamped for reads; stores are masked), chunk 0 into buffer 0,
  // weights of steps 0 .. kW - 2.  The groups take turns at bringing in a chunk: chunk kc is group kc mod
  // KG's, which asks for its next one as soon as it has put one into LDS.
  // (lane -> channel co_w + lane of the wave's 16 NT)
  unsigned char* const consts = xs + 3 * bufbytes + wave * 768;   // [m, s, bias][64] of this wave's channels
  if (kg == 0) {
    const int64_t co = min(co_w + (lane & (16 * NT - 1)), p.Cout - 1);
    direct_load4(p.m + co, consts);
    direct_load4(p.s + co, consts + 256);
    if (p.bias) direct_load4(p.bias + co, consts + 512);
  }
  if (kg == 0) issue_chunk(0);
#pragma unroll
  for (int u = 0; u < kW - 1; ++u) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) load_w(nt, wb[u]);
    next_w();
  }
  int xcnt = 0;                                     // steps whose weights were requested before the chunk on its way
  wait_vm<(kW - 1) * NT>();
  v4i acc[MT][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = (v4i){0, 0, 0, 0};
  if (kg == 0) commit_chunk(0);
  if ((kg == 0 ? KG : kg) < nkc) {
    issue_chunk(kg == 0 ? KG : kg);
    xcnt = kW - 1;
  }
  __syncthreads();

  // The A operands (one 16-byte LDS read per 16 frames) go through a ring of four registers, three reads
  // ahead of the products, across steps and chunks: chunk kc + 1 is complete in LDS from the middle of chunk
  // kc on (three buffers, one barrier per chunk: the wave that puts chunk kc + 1 where chunk kc - 2 was has
  // passed the barrier in the middle of chunk kc - 1, which no wave reaches before it is done with kc - 2).
  auto arow_of = [&](int buf_, int j_) __attribute__((always_inline)) {
    return xs + buf_ * bufbytes + (foff + j_ * p.dil + n * p.stride) * kXS + 16 * gi;
  };
  auto read_a = [&](const unsigned char* arow, int mt) __attribute__((always_inline)) {
    return *reinterpret_cast<const v4i*>(arow + 16 * mt * p.stride * kXS);
  };
  const int jmid = j0 + ((j1 - j0) >> 1);           // the tap before which the next chunk is committed
  int kc = 0, j = j0, buf = 0, q = 0;               // chunk, tap and buffer of the current step
  const unsigned char* arow = arow_of(0, j0);
  v4i ar[4];
  ar[0] = read_a(arow, 0);
  ar[1] = read_a(arow, 1);
  ar[2] = read_a(arow, 2);
  auto step = [&](auto slot_tag) __attribute__((always_inline)) {
    constexpr int u = decltype(slot_tag)::value;
    if (j == jmid && kc + 1 < nkc) {
      const int nbuf = buf == 2 ? 0 : buf + 1;
      if (KG == 1 || kg == (kc + 1) % KG) {
        // (3 - xcnt steps' weights were requested after the chunk, more if xcnt is 0)
        if (xcnt == 3) wait_vm<0>();
        else if (xcnt == 2) wait_vm<NT>();
        else wait_vm<2 * NT>();
        commit_chunk(nbuf);
        if (kc + 1 + KG < nkc) {
          issue_chunk(kc + 1 + KG);
          xcnt = kW - 1;
        }
      }
      __syncthreads();                              // chunk kc + 1 is in LDS
    }
    // this step's weights: those of the kW - 2 steps after it are younger, and so may a chunk's 16 dwords be
    if (xcnt > 0) {
      --xcnt;
      wait_vm<(kW - 2) * NT + 16>();
    } else {
      wait_vm<(kW - 2) * NT>();
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) tie(wb[u][nt]);
    if (++j == j1) {
      if (kc + 1 < nkc) { j = j0; ++kc; buf = buf == 2 ? 0 : buf + 1; }
      else --j;                                     // (after the last step: the operands are read once more)
    }
    const unsigned char* const anext = arow_of(buf, j);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      ar[(u * MT + mt + 3) % 4] = mt + 3 < MT ? read_a(arow, mt + 3) : read_a(anext, mt + 3 - MT);
      if (mt < NT) load_w(mt, wb[(u + kW - 1) % kW]);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
        acc[mt][nt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ar[(u * MT + mt) % 4], wb[u][nt], acc[mt][nt], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    next_w();
    arow = anext;
    return ++q < Q;
  };
  static_assert(kW == 4 && MT >= NT && MT >= 3, "rings");
  while (step(std::integral_constant<int, 0>{}) && step(std::integral_constant<int, 1>{}) &&
         step(std::integral_constant<int, 2>{}) && step(std::integral_constant<int, 3>{})) {}
  wait_vm<0>();                                     // what the weight stream asked for past its end
#pragma unroll
  for (int u = 0; u < kW; ++u)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) tie(wb[u][nt]);

  // ---- KG > 1: group o finishes the frame groups mt with mt KG / MT == o; every other group's sums of
  // them reach it through LDS (past the activation buffers: no wave may be reading those any more)
  if constexpr (KG > 1) {
    static_assert(MT % KG == 0, "frame groups per wave group");
    // [owner][the other groups][frame group of the owner][nt][wave][lane]
    v4i* const red = reinterpret_cast<v4i*>(xs + 3 * bufbytes + kConstBytes);
    auto slot = [&](int o, int src, int mt, int nt) __attribute__((always_inline)) {
      const int rank = src < o ? src : src - 1;
      return red + ((((o * (KG - 1) + rank) * (MT / KG) + mt % (MT / KG)) * NT + nt) * 4 + wave) * 64 + lane;
    };
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      if (mt * KG / MT != kg) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) *slot(mt / (MT / KG), kg, mt, nt) = acc[mt][nt];
      }
    __syncthreads();
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      if (mt * KG / MT == kg) {
#pragma unroll
        for (int o = 1; o < KG; ++o) {
          const int src = (kg + o) % KG;
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) acc[mt][nt] += *slot(kg, src, mt, nt);
        }
      }
  }

  // ---- splits > 1 (a launch of few tiles would leave most compute units idle while each of its
  // workgroups goes through the whole contraction: 768 channels, 25 taps, 2 x 200 frames 50 -> 20 us
  // with four): the sums of this range go to memory, and the workgroup of the tile that comes last
  // adds those of the others to its own and goes on.  The handover is release and acquire at device scope,
  // which on this chip is what makes one die's writes appear behind another die's L2: every wave's stores
  // are complete before the barrier, thread 0 counts the arrival with release order (what its L2 still holds
  // of them is written back), and the thread that finds itself last makes the acquire fence (its die's
  // stale lines go) before the barrier behind which the others' sums are loaded.  Nobody waits for anybody.
  // (Dense-residual Jasper, 2 x 811 frames: 1366 us; 1487 with write-back stores; 1278 with a relaxed count and
  // loads past the caches, an order that nothing promises; of the 88 us the write-back is 62, the fence 26.)
  if (g.splits > 1) {
    auto part_of = [&](int s_) __attribute__((always_inline)) {
      return __builtin_amdgcn_make_buffer_rsrc(p.part + ((int64_t)(co_tile * nbt + bt) * g.splits + s_) * (MT * NT * 1024), 0,
                                               MT * NT * 4096, 0x00027000);
    };
    const uint32_t poff = (uint32_t)(wave * 64 + lane) * 16;
    auto owned = [&](int mt) { return KG == 1 || mt * KG / MT == kg; };
    const __amdgpu_buffer_rsrc_t mine = part_of(split);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      if (owned(mt)) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, acc[mt][nt]), mine, poff, (mt * NT + nt) * 4096, kStoreThrough);
      }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();                                // (the LDS buffers have been read by all, too)
    if (threadIdx.x == 0) {
      unsigned* const count = p.part_count + co_tile * nbt + bt;
      const unsigned before = __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
      if (before + 1 == (unsigned)g.splits) {
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        __hip_atomic_store(count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // (for the next layer)
      }
      *reinterpret_cast<volatile unsigned*>(xs) = before;
    }
    __syncthreads();
    if (*reinterpret_cast<volatile unsigned*>(xs) + 1 != (unsigned)g.splits) return;   // whole workgroup
    // (the sums of several ranges on their way at once where a wave has few of them)
    constexpr int OB = MT * NT / KG <= 4 ? 4 : 1;
#pragma unroll 1
    for (int o0 = 1; o0 < g.splits; o0 += OB) {
      v4i in[OB][MT * NT / KG];
#pragma unroll
      for (int i = 0; i < OB; ++i) {
        const int o = split + min(o0 + i, g.splits - 1);   // (past the last range: loaded again, not added)
        const __amdgpu_buffer_rsrc_t from = part_of(o < g.splits ? o : o - g.splits);
#pragma unroll
        for (int j = 0; j < MT * NT / KG; ++j)
          in[i][j] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(from, poff, (kg * (MT * NT / KG) + j) * 4096, 0));
      }
#pragma unroll
      for (int i = 0; i < OB; ++i)
        if (o0 + i < g.splits) {
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
            if (owned(mt)) {
#pragma unroll
              for (int nt = 0; nt < NT; ++nt) acc[mt][nt] += in[i][mt % (MT / KG) * NT + nt];
            }
        }
    }
  }

  // ---- epilogue: lane (n, gi) holds frames t0 + 16 mt + 4 gi + (0..3) of channel co_w + 16 nt + n
  constexpr int NB = MT / KG;                       // frame groups that this wave finishes: kg NB + h
  const int trow = p.Tout + p.ypad;                 // (pad bytes may be written)
  const int tl = t0 + 16 * NB * kg + 4 * gi;
  const int64_t orow = (int64_t)b * p.ybs + (int64_t)(co_w + n) * trow;
  v4i fin[NB][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
    if (KG == 1 || mt / NB == kg) {
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) fin[mt % NB][nt] = acc[mt][nt];
    }
  bool on[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    on[nt] = co_w + 16 * nt + n < p.Cout;
    const int32_t* const cl = reinterpret_cast<const int32_t*>(consts) + 16 * nt + n;
    const int32_t mc = cl[0], sc = cl[64], bv = p.bias ? cl[128] : 0;
#pragma unroll
    for (int h = 0; h < NB; ++h)
#pragma unroll
      for (int i = 0; i < 4; ++i) fin[h][nt][i] = dyadic_rescale(fin[h][nt][i] + bv, mc, sc);
  }
  // residual operands (dense-residual layers have several): the rows of RB of them on their way at once
  if (p.res) {
    constexpr int RB = NB * NT <= 4 ? 6 : NB * NT <= 10 ? 3 : 2;
    const int count = 1 + p.n_res_more;
#pragma unroll 1
    for (int r0 = 0; r0 < count; r0 += RB) {
      uint32_t d[RB][NB][NT];
#pragma unroll
      for (int r = 0; r < RB; ++r)
        if (r0 + r < count) {                       // (uniform)
          const int8_t* const src = (r0 + r == 0 ? p.res : p.res_more[r0 + r - 1]) + orow;
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int h = 0; h < NB; ++h) {
              const int t = tl + 16 * h;
              d[r][h][nt] = 0;
              if (on[nt] && t < p.Tout) d[r][h][nt] = load_u32(src + (int64_t)(16 * nt) * trow + min(t, trow - 4));
            }
        }
#pragma unroll
      for (int r = 0; r < RB; ++r)
        if (r0 + r < count) {
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int h = 0; h < NB; ++h) {
              const int t = tl + 16 * h;
              const uint32_t w = t > trow - 4 ? d[r][h][nt] >> (8 * (t - (trow - 4))) : d[r][h][nt];   // (load_row_u32)
#pragma unroll
              for (int i = 0; i < 4; ++i) fin[h][nt][i] += (int32_t)(int8_t)(w >> (8 * i));
            }
        }
    }
  }
  const int lo = p.relu ? 0 : -128;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int h = 0; h < NB; ++h) {
      const int t = tl + 16 * h;
      if (!on[nt] || t >= p.Tout) continue;
      uint32_t pk = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) pk |= (uint32_t)(clamp_i8(fin[h][nt][i], lo) & 0xff) << (8 * i);
      store_row_u32(p.y + orow + (int64_t)(16 * nt) * trow, t, trow, pk);
    }
}

int lds_rows(const ConvParams& p, int TM) {
  // frames read by a tile: (TM-1)*stride + dil*(k-1) + 1, plus up to 3 of dword alignment slack
  return (((TM - 1) * p.stride + p.dil * (p.k - 1) + 1 + 3) + 3) & ~3;
}

struct CpTile { int MT, NT, KG, S; };

constexpr int64_t kMaxSplitTiles = kConvSplitCounters;   // (one arrival counter each)

size_t lds_bytes(const ConvParams& p, const CpTile& c) {
  const size_t x = (size_t)3 * lds_rows(p, 16 * c.MT) * kXS + kConstBytes;
  return c.KG > 1 ? x + (size_t)(c.KG - 1) * c.MT * c.NT * 4096 : x;
}

// Workgroups of a tile that a compute unit holds: registers (512 per SIMD and lane), then LDS.
int resident(const ConvParams& p, const CpTile& c) {
  const int by_regs = c.KG == 4 ? 1 : c.KG == 2 ? (c.MT * c.NT <= 8 ? 2 : 1) : c.NT == 4 || c.MT > 9 ? 2 : c.MT > 4 ? 3 : 4;
  const int by_lds = (int)(160 * 1024 / lds_bytes(p, c));
  return by_regs < by_lds ? by_regs : by_lds;
}

// Cycles that a compute unit takes for n workgroups of a tile whose contraction is `chunks` chunks long.  w of them
// run at once: a step is bound by the matrix pipes (18.6 cycles per product: with operands that are not zeros the
// clock gives way), by a lone wave's own latencies, by the weights (NT KiB per wave) or by the operand reads; a
// chunk costs a commit and a barrier; a workgroup its first loads and its epilogue, KG > 1 the meeting of the sums.
// The constants are fitted to chains of six layers whose weights are in no L2.  Every tile, with 1, 2, 3, 4, 6 and 8
// splits where the launch is small, timed beside the choice: 256 .. 768 channels, 11 .. 25 taps, 52 .. 12800 frames, 60
// shapes: it is 0.4 % from the best on average and 8.0 % at worst (384 channels, 2 x 800 frames).
double unit_cycles(const ConvParams& p, const CpTile& c, int64_t n, int chunks) {
  const double mn = c.MT * c.NT, taps = (p.k + c.KG - 1) / c.KG;
  const int occ = resident(p, c);
  auto T = [&](int64_t w) {
    if (w == 0) return 0.0;
    const double step = fmax(fmax(18.6 * (double)w * c.KG * mn, 16.0 * mn + 343.0),
                             fmax(93.0 * (double)w * c.KG * c.NT, 29.0 * (double)w * c.KG * c.MT));
    return 3900.0 + 690.0 * mn / c.KG * (double)w + chunks * (fmax(taps * step, 890.0) + 920.0) + (c.KG > 1 ? 7800.0 : 0.0);
  };
  return (double)(n / occ) * T(occ) + T(n % occ);
}

bool pick(const ConvParams& p, bool split, CpTile& best_tile, double& best) {
  if (tuning().no_conv_pipe) return false;                // tuning: fall through to gemm_mfma
  if (p.depthwise || p.Cin % 64 != 0 || !p.w_packed || p.k < 2) return false;
  if (p.Cout < 64) return false;
  if (p.Tin < 4 || p.Tout < 4 || (uintptr_t)p.w % 16) return false;   // (rows are read in dwords, at any address)
  // the kernel addresses the packed weights with 32-bit offsets
  if ((int64_t)p.k * ((p.Cout + 15) / 16) * (p.Cin / 64) * 1024 > 0x7fffffffLL) return false;
  const int force_mt = tuning().cp_mt, force_nt = tuning().cp_nt, force_kg = tuning().cp_kg;   // tuning
  static const CpTile tiles[] = {{8, 4, 1, 1}, {7, 4, 1, 1}, {6, 4, 1, 1}, {5, 4, 1, 1}, {4, 4, 1, 1}, {10, 2, 1, 1}, {9, 2, 1, 1}, {8, 2, 1, 1}, {7, 2, 1, 1}, {6, 2, 1, 1},
                                 {5, 2, 1, 1}, {4, 2, 1, 1}, {6, 4, 2, 1}, {4, 4, 2, 1}, {10, 2, 2, 1}, {8, 2, 2, 1}, {6, 2, 2, 1}, {4, 2, 2, 1}, {4, 2, 4, 1}};
  const int force_s = tuning().cp_s;
  best = 1e300;
  bool found = false;
  for (const CpTile& c : tiles) {
    if ((force_mt && c.MT != force_mt) || (force_nt && c.NT != force_nt) || (force_mt && c.KG != (force_kg ? force_kg : 1))) continue;
    if (c.KG > p.k || lds_bytes(p, c) > 160 * 1024) continue;
    const int TM = 16 * c.MT;
    const int rows = lds_rows(p, TM);
    if (rows > kMaxRows || (int64_t)p.Cin * (p.Tin + p.xpad) > 0x7fffffffLL) continue;
    const int64_t n_tt = (p.Tout + TM - 1) / TM, n_co = (p.Cout + 64 * c.NT - 1) / (64 * c.NT);
    const int64_t blocks = (int64_t)p.B * n_tt * n_co;
    if (blocks > 0x7ffffff0LL) continue;
    for (int S = 1; S <= (split && blocks <= kMaxSplitTiles ? kMaxSplits : 1) && S <= p.Cin / 64; ++S) {
      if (force_s && split && S != force_s) continue;
      // the longest range of chunks; the other splits' sums read back one after the other, and all sums through memory
      const int64_t wgs = blocks * S;
      const double cost = unit_cycles(p, c, (wgs + 255) / 256, (p.Cin / 64 + S - 1) / S) +
                          (S > 1 ? 10700.0 + 1445.0 * (S - 1) + c.MT * c.NT / (double)c.KG * (9.3 * (S - 1) + 4.0 * (double)wgs) : 0.0);
      if (cost < best * 0.999) { best = cost; best_tile = c; best_tile.S = S; found = true; }
    }
  }
  return found;
}

size_t part_bytes(const ConvParams& p, const CpTile& c) {
  if (c.S == 1) return 0;
  const int64_t n_tt = (p.Tout + 16 * c.MT - 1) / (16 * c.MT), n_co = (p.Cout + 64 * c.NT - 1) / (64 * c.NT);
  return (size_t)(p.B * n_tt * n_co) * c.S * (c.MT * c.NT * 4096);
}

__global__ __launch_bounds__(kConvSplitCounters) void conv_split_clear_kernel(unsigned* counters) { counters[threadIdx.x] = 0; }

template <int MT, int NT, int KG>
hipError_t launch_t(const ConvParams& p, int splits, hipStream_t st) {
  constexpr int TM = 16 * MT, TN = 64 * NT;
  CpGeom g;
  g.n_tt = (p.Tout + TM - 1) / TM;
  g.n_co = (p.Cout + TN - 1) / TN;
  g.rows = lds_rows(p, TM);
  g.kchunks = p.Cin / 64;
  g.co16n = (p.Cout + 15) / 16;
  g.splits = splits;
  const int64_t blocks = (int64_t)p.B * g.n_tt * g.n_co * splits;
  g.tiles = (int)blocks;
  g.per_xcd = tuning().cp_plain_order ? 0 : (int)((blocks + 7) / 8);
  g.r_nbt = 1.0f / (float)(p.B * g.n_tt);
  g.r_splits = 1.0f / (float)splits;
  g.r_tt = 1.0f / (float)g.n_tt;
  g.fq_inv = (65536 + g.rows / 4 - 1) / (g.rows / 4);
  const size_t lds = lds_bytes(p, CpTile{MT, NT, KG, 1});
  if (lds > 64 * 1024) {
    static std::atomic<uint64_t> lds_raised{0};   // per instantiation, a bit per device
    if (const hipError_t e = ensure_max_dynamic_lds((const void*)conv_pipe_kernel<MT, NT, KG>, lds_raised); e != hipSuccess)
      return e;
  }
  return launch_kernel(conv_pipe_kernel<MT, NT, KG>, dim3((unsigned)(g.per_xcd ? 8 * g.per_xcd : (int)blocks)), dim3(256 * KG),
                       lds, st, p, g);
}

}  // namespace

bool conv_pipe_supported(const ConvParams& p) {
  CpTile c;
  double t;
  return pick(p, false, c, t);
}

bool conv_few_better(const ConvParams& p, bool split, FewTile& tile) {
  CpTile c;
  double few, pipe;
  if (tuning().cp_mt || !conv_few_cycles(p, tile, few)) return false;
  return tuning().conv_few_force || !pick(p, split, c, pipe) || few < pipe;
}

size_t conv_pipe_split_bytes(const ConvParams& p) {
  CpTile c;
  FewTile few;
  double t;
  return pick(p, true, c, t) && !conv_few_better(p, true, few) ? part_bytes(p, c) : 0;
}

hipError_t launch_conv_split_clear(unsigned* counters, hipStream_t st) {
  return launch_kernel(conv_split_clear_kernel, dim3(1), dim3(kConvSplitCounters), 0, st, counters);
}

hipError_t launch_conv_pipe(const ConvParams& p, hipStream_t st) {
  CpTile c;
  double t;
  bool ok = pick(p, p.part != nullptr, c, t);
  if (!ok || (int64_t)part_bytes(p, c) > p.part_bytes) ok = pick(p, false, c, t);   // (tuning changed since the room was made)
  if (!ok) return hipErrorInvalidValue;
#define QASR_CASE(M, N, K) if (c.MT == M && c.NT == N && c.KG == K) return launch_t<M, N, K>(p, c.S, st);
  QASR_CASE(8, 4, 1) QASR_CASE(7, 4, 1) QASR_CASE(6, 4, 1) QASR_CASE(5, 4, 1) QASR_CASE(4, 4, 1) QASR_CASE(10, 2, 1) QASR_CASE(9, 2, 1)
  QASR_CASE(8, 2, 1) QASR_CASE(7, 2, 1) QASR_CASE(6, 2, 1) QASR_CASE(5, 2, 1) QASR_CASE(4, 2, 1)
  QASR_CASE(6, 4, 2) QASR_CASE(4, 4, 2) QASR_CASE(10, 2, 2) QASR_CASE(8, 2, 2) QASR_CASE(6, 2, 2) QASR_CASE(4, 2, 2) QASR_CASE(4, 2, 4)
#undef QASR_CASE
  return hipErrorInvalidValue;
}

}  // namespace qasr
