// Planning and launching of the fused separable module (sep_body.hpp), and the weight image its depthwise
// half multiplies with.
#include "launch_shape.hpp"
#include "sep_body.hpp"
#include "tuning.hpp"

namespace qasr {

namespace {

struct Geometry { int delta, r, nk, NA; };

bool geometry(const ConvParams& d, Geometry& g) {
  if (!d.depthwise || d.stride != 1 || d.res || d.n_res_more || d.Tout < 1) return false;
  g.delta = ((-d.pl) % 16 + 16) % 16;                    // rows are loaded from a multiple of 16 frames
  g.r = g.delta & 3;                                     // (whole dwords of it are an address offset)
  const int64_t span = (int64_t)d.dil * (d.k - 1) + 1;
  if (span > 96) return false;
  g.nk = (int)((span + 3 + g.r + 3) / 4);
  g.NA = g.nk <= 12 ? 3 : (g.nk + 3) / 4;
  return g.NA <= 6;
}

// rows that start at 16-byte boundaries and are padded to them are moved in whole chunks
bool x_ragged(const ConvParams& d) { return (d.Tin + d.xpad) % 16 || d.xbs % 16 || (uintptr_t)d.x % 16; }
bool y_ragged(const ConvParams& q) {
  return (q.Tout + q.ypad) % 16 || q.ybs % 16 || (uintptr_t)q.y % 16 || (uintptr_t)q.res % 16;
}

int units_of(const ConvParams& d, const Geometry& g, int MT) {
  const int need = (g.delta + 16 * MT + d.dil * (d.k - 1) + 15) / 16;
  return need | 1;
}

// The weights as the kernels load them: rows [C][16 NA bytes], tap j at byte r + j dil, zeros between and after the last.
size_t weight_bytes(int C, int NA) { return (size_t)C * NA * 16; }
size_t image_bytes(int C, int NA) { return weight_bytes(C, NA) + DwParams::kImageTail; }
__global__ __launch_bounds__(256) void sep_image_kernel(const int8_t* __restrict__ w, int C, int k, int dil, int r, int NA,
                                                        uint32_t* __restrict__ rows) {
  const int idx = (int)(blockIdx.x * blockDim.x + threadIdx.x), c = idx / (4 * NA);
  if (idx >= C * NA * 4 + DwParams::kImageTail / 4) return;
  uint32_t v = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int rel = 4 * (idx % (4 * NA)) - r + e, j = rel >= 0 ? rel / dil : -1;
    if (c < C && j >= 0 && j < k && j * dil == rel) v |= (uint32_t)(uint8_t)w[(int64_t)c * k + j] << (8 * e);
  }
  rows[idx] = v;
}

size_t lds_bytes(int KCH, int units, int MT, int NA, int NT, int KS) {
  const int rows = MT <= 2 ? sep::small_row_bytes(4 * KCH, sep::row_units(MT, NA), MT, NA) : sep::row_bytes(units, MT, NA);
  return (size_t)KCH * 8192 + sep::kWaves * (size_t)(rows + 256) + (MT <= 2 ? 12 * (size_t)(256 / KS * NT) : 0);
}

// Tile (MT groups x 256 NT output channels per workgroup) with the least time on the busiest compute
// unit, one workgroup at a time: its matrix pipes (10 cycles per 4x4x4 product, 17.7 per 16x16x64 one),
// its 64 bytes per cycle from the L2 (weight rows and packed weights, which every workgroup streams whole, and rows), and the
// latency of its first loads and last stores.  With a projection there are as many workgroups again, without the depthwise
// half: a list, in which one costs less where two fit on a unit (256 channels) or each has half a tile's products.
// Every tile timed beside the choice (profiles/pair_tile_choice.txt), weights in no L2 as in a network: 320 pairs and 320 with
// projection, of 256 or 512 channels, 33 to 87 taps, 32 to 26000 frames.  The choice is 0.2 and 1.1 % from the best on average, 9 and
// 28 % at worst (256 channels, 33 taps, 14 x 1034 frames: of a pair it knows of no two workgroups on a unit).  With the weight rows at four
// times their bytes, as when they were a prebuilt operand, all bytes half hidden and 5.0 for every list, it was 0.6 and 5.9 % from it.
bool pick(const ConvParams& d, const ConvParams& q, const Geometry& g, int groups_per_row, int cus, bool proj, SepChoice& c) {
  static const int MTs[] = {1, 2, 4, 7};
  c.KCH = d.Cout / 64;
  c.NA = g.NA;
  double best = 1e300;
  const int force_mt = tuning().sep_mt, force_nt = tuning().sep_nt, force_ks = tuning().sep_ks;
  for (int KS = 1; KS <= 2; ++KS) {
    for (int NT = 1; NT <= 2; ++NT) {
      if (q.Cout % (256 / KS * NT) || (force_nt && NT != force_nt)) continue;
      for (int MT : MTs) {
        if ((force_mt && MT != force_mt) || (c.ragged && MT > 4)) continue;
        if ((KS > 1 && (MT > 2 || NT > 1)) || (force_nt && (force_ks ? force_ks : 1) != KS)) continue;
        const int units = units_of(d, g, MT);
        if (units > sep::kMaxUnits) continue;
        if (MT <= 2 && (int64_t)4 * c.KCH * (d.Tin + d.xpad) > 0x7fffffffLL) continue;   // 32-bit offsets within a wave's rows
        const size_t lds = lds_bytes(c.KCH, units, MT, c.NA, NT, KS);
        if (lds > 160 * 1024) continue;
        const int splits = q.Cout / (256 / KS * NT);
        const int64_t wgs = (int64_t)d.B * ((groups_per_row + MT - 1) / MT) * splits;
        if (wgs * (proj ? 2 : 1) > max_workgroups(64 * sep::kWaves) || wgs * ((groups_per_row + MT - 1) / MT) > 1LL << 32) continue;   // (place)
        const double mfma = c.KCH / 2 * MT * g.nk * 10.0 * 2 + MT * NT * c.KCH * 17.7 * 4 / KS;
        const double bytes = (double)weight_bytes(d.Cout, c.NA) + NT * 16.0 * c.KCH * 1024 / KS + c.KCH * 64.0 * units * 16;
        const double work = (mfma + bytes / 64) / 2200.0 + 1.0 + 0.1 * MT * NT;
        const int64_t n = (wgs + cus - 1) / cus;
        double cost = (double)n * (2.5 + work);
        if (proj) {                                 // as many workgroups again, without the depthwise half: as a list
          const double each = c.KCH == 4 ? 4.5 : KS == 2 ? 5.0 : 8.0;
          const double work2 = (MT * NT * c.KCH * 17.7 * 4 / KS + (NT * 16.0 * c.KCH * 1024 / KS + c.KCH * 1024.0 * MT) / 64) / 2200.0 + 1.0 + 0.1 * MT * NT;
          const double list = (double)wgs * (each + work + work2) / cus;
          if (list > cost) cost = list;
        }
        if (cost < best) { best = cost; c.MT = MT; c.NT = NT; c.KS = KS; c.splits = splits; }
      }
    }
  }
  return best < 1e300;
}

bool plan(const ConvParams& d, const ConvParams& q, int cus, bool proj, Geometry& g, SepChoice& c) {
  if (tuning().no_sep || !geometry(d, g)) return false;
  if (d.Cout != 256 && d.Cout != 512) return false;
  if (q.depthwise || q.k != 1 || q.stride != 1 || q.pl != 0 || !q.w_packed || q.Cin != d.Cout || q.n_res_more || q.act_lut)
    return false;
  if (q.Cout % 256 || q.Cout > 2048 || (uintptr_t)q.w % 16) return false;
  if (q.Tout != q.Tin) return false;                     // (padded on the right: it reads zeros there, not what the tile holds)
  if (d.Tout != q.Tin && (d.Tout + 15) / 16 * 16 != q.Tin) return false;            // (q may run over the pitch)
  // 32-bit offsets within 16 rows of x and a batch item of y
  if ((int64_t)16 * (d.Tin + d.xpad) > 0x7fffffffLL || (int64_t)q.Cout * (q.Tout + q.ypad) > 0x7fffff00LL) return false;
  if (d.xbs >= 1LL << 32 || q.ybs >= 1LL << 32) return false;
  if (d.Tin < 4 || q.Tout < 4) return false;
  c.ragged = x_ragged(d) || y_ragged(q);
  return pick(d, q, g, (q.Tout + 15) / 16, cus, proj, c);
}

}  // namespace

bool sep_choice(const ConvParams& d, const ConvParams& q, bool projection, SepChoice& c) {
  Geometry g;
  return plan(d, q, 256, projection, g, c);
}
bool sep_supported(const ConvParams& d, const ConvParams& q) {
  SepChoice c;
  return sep_choice(d, q, false, c);
}

// Wherever it can: blocks of a projection and a pair, 256 or 512 -> 256 .. 2048 channels, 1 x 104 .. 64 x 800 frames, take
// 0.69 to 1.01 of their time apart (80 shapes; above 0.98 at 64 x 800 and, of 512 -> 2048, 32 x 800, where a launch is nothing).
bool sep_projection_supported(const ConvParams& d, const ConvParams& q, const ConvParams& r) {
  Geometry g;
  SepChoice c;
  if (!plan(d, q, 256, true, g, c) || c.ragged) return false;
  if ((int64_t)32 * (d.Tin + d.xpad) > 0x7fffffffLL) return false;   // 32-bit offsets within a wave's rows of the tile
  return !r.depthwise && r.k == 1 && r.stride == 1 && r.pl == 0 && r.Tout == r.Tin && r.w_packed && !r.res && !r.n_res_more && !r.act_lut &&
         r.B == d.B && r.Cin == d.Cin && r.Cout == q.Cout && r.xbs == d.xbs && r.Tin + r.xpad == d.Tin + d.xpad && r.ybs == q.ybs &&
         r.Tout + r.ypad == q.Tout + q.ypad && (r.Tout + 15) / 16 == (q.Tout + 15) / 16 && (uintptr_t)r.w % 16 == 0 &&
         (uintptr_t)r.y % 16 == 0 && r.x == d.x;
}

static void fill_dw(const ConvParams& d, const Geometry& g, int MT, DwParams& p) {
  p.x = d.x; p.dbias = d.bias; p.dm = d.m; p.ds = d.s; p.lut = d.act_lut;
  p.xbs = d.xbs; p.xpitch = d.Tin + d.xpad; p.Tin = d.Tin;
  p.o16 = -((d.pl + g.delta) / 16);
  p.nk = g.nk;
  p.units = units_of(d, g, MT);
  p.dwoff = g.delta >> 2;
  p.drelu = d.relu;
  p.units_inv = (65536 + p.units - 1) / p.units;
  const int need = (g.delta + 16 * MT + d.dil * (d.k - 1) + 15) / 16;
  p.row_lanes_log2 = need > 8 ? 4 : need > 4 ? 3 : 2;
  p.row_step = (int32_t)((64 >> p.row_lanes_log2) * (int64_t)p.xpitch);
}

bool dw_small_params(const ConvParams& d, int MT, DwParams& p, int& NA) {
  Geometry g;
  if (!geometry(d, g) || MT > 2 || d.Cout % 256 || d.Tin < 4 || x_ragged(d)) return false;
  fill_dw(d, g, MT, p);
  NA = g.NA;
  const int C = d.Cout / sep::kWaves;               // rows a wave brings in at a time
  return p.units <= sep::kMaxUnits && (int64_t)C * p.xpitch <= 0x7fffffffLL && C * p.units <= 64 * sep::row_loads(C, MT, NA);
}

size_t sep_image_bytes(const ConvParams& d) {
  Geometry g;
  return geometry(d, g) ? image_bytes(d.Cout, g.NA) : 0;
}

hipError_t launch_sep_image(const ConvParams& d, uint32_t* img, hipStream_t st) {
  Geometry g;
  if (!geometry(d, g) || d.Cout % 16) return hipErrorInvalidValue;
  return launch_kernel(sep_image_kernel, dim3((unsigned)((image_bytes(d.Cout, g.NA) / 4 + 255) / 256)), dim3(256), 0, st, d.w, d.Cout, d.k, d.dil, g.r,
                       g.NA, img);
}

static hipError_t launch(const ConvParams& d, const uint32_t* img, const ConvParams& q, const ConvParams* r, hipStream_t st) {
  Geometry g;
  SepChoice c;
  if (!plan(d, q, compute_units(), r != nullptr, g, c)) return hipErrorInvalidValue;
  SepParams p{};
  fill_dw(d, g, c.MT, p);
  p.img = img;
  p.pw[0] = {q.w, q.bias, q.m, q.s, q.res, q.y, q.relu, 0};
  if (r) p.pw[1] = {r->w, r->bias, r->m, r->s, nullptr, r->y, r->relu, 0};
  p.ybs = q.ybs; p.ypitch = q.Tout + q.ypad; p.Tout = q.Tout;
  const int gpr = (q.Tout + 15) / 16;
  p.tpr = (gpr + c.MT - 1) / c.MT;
  p.g_base = gpr / p.tpr;
  p.g_more = gpr % p.tpr;
  p.yragged = y_ragged(q);
  p.splits = c.splits;
  p.wgs = d.B * p.tpr * p.splits;                // (< 2^22: pick)
  p.splits_inv = 0xffffffffu / (uint32_t)p.splits;
  p.tpr_inv = 0xffffffffu / (uint32_t)p.tpr;
  if (c.MT > 2 && 16 * p.units > 64 * sep::row_loads(16, c.MT, c.NA)) return hipErrorInvalidValue;
  p.per_xcd = (p.wgs + 7) / 8;
  const size_t lds = lds_bytes(c.KCH, p.units, c.MT, c.NA, c.NT, c.KS);
  switch (c.NA) {
    case 3: return launch_sep_na3(c, p, lds, st);
    case 4: return launch_sep_na4(c, p, lds, st);
    case 5: return launch_sep_na5(c, p, lds, st);
    default: return launch_sep_na6(c, p, lds, st);
  }
}

hipError_t launch_sep(const ConvParams& d, const uint32_t* img, const ConvParams& q, hipStream_t st) {
  return launch(d, img, q, nullptr, st);
}
hipError_t launch_sep(const ConvParams& d, const uint32_t* img, const ConvParams& q, const ConvParams& r, hipStream_t st) {
  if (!sep_projection_supported(d, q, r)) return hipErrorInvalidValue;
  return launch(d, img, q, &r, st);
}

}  // namespace qasr
