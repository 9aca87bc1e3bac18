// A depthwise layer and the pointwise layer that reads it as one launch (the separable module of the
// QuartzNet family, the convolution module's tail of the Conformer): what sep.hip plans and launches and
// sep_body.hpp computes.
#pragma once
#include "common.hpp"

#include <cstddef>

namespace qasr {

// a depthwise layer whose output stays in LDS
struct DwParams {
  // x rows (pitch xpitch, batch stride xbs, Tin frames), weights (sep.hip: image)
  const int8_t* x;
  const uint32_t* img;
  static constexpr int kImageTail = 1024;   // bytes of zeros after the weights, into which a wave's last load may run
  const int32_t *dbias, *dm, *ds;    // dbias may be null
  const uint8_t* lut;                // table of a unary activation between the two layers, or null
  int64_t xbs;
  int32_t xpitch, Tin;
  int32_t o16;                       // first chunk of a tile's rows relative to its first frame: (-pl - delta) / 16
  int32_t nk;                        // 4-tap steps
  int32_t units;                     // 16-byte chunks per row in LDS (odd: 16 rows then start in different banks)
  int32_t dwoff;                     // dwords between a row's start and the first window
  int32_t drelu;
  int32_t units_inv;                 // ceil(2^16 / units): L / units = L units_inv >> 16 for L < 512, units <= 15
  int32_t row_lanes_log2, row_step;  // small tiles: lanes that bring a row in; bytes between the first rows of two requests
};

struct SepPointwise {
  const int8_t* w;                   // packed (common.hpp)
  const int32_t *bias, *m, *s;       // bias may be null
  const int8_t* res;                 // may be null
  int8_t* y;
  int32_t relu, pad_;
};
struct SepParams : DwParams {
  // pointwise half: [0] the pair's; [1] a second pointwise layer of x itself (a block's residual projection), by workgroups of its
  // own in the same launch (blockIdx.z): widths, rows and tiles of the first, no residual
  SepPointwise pw[2];
  int64_t ybs;                       // both batch strides < 2^32
  int32_t ypitch;
  int32_t Tout, yragged;             // frames per row; rows (y and residual) not padded to whole aligned chunks
  // tiles: the 16-frame groups of a row (batch item) make tpr tiles of g_base groups, the first g_more of them
  // one group more
  int32_t tpr, g_base, g_more;
  int32_t splits;                    // workgroups per tile, each with its own run of output channels
  int32_t wgs, per_xcd;              // workgroups in all (of one layer), and per XCD
  uint32_t splits_inv, tpr_inv;      // (2^32 - 1) / the two: v / d = (v + 1) inv >> 32 while (v + 1) d <= 2^32
};

// the kernels read these in pairs (sep_body.hpp: and_next)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winvalid-offsetof"
#define QASR_NEIGHBOURS(a, b) static_assert(offsetof(SepParams, b) == offsetof(SepParams, a) + 4, #a " and " #b " are read as one")
QASR_NEIGHBOURS(ypitch, Tout);
QASR_NEIGHBOURS(yragged, tpr);
QASR_NEIGHBOURS(g_base, g_more);
QASR_NEIGHBOURS(splits, wgs);
QASR_NEIGHBOURS(xpitch, Tin);
QASR_NEIGHBOURS(o16, nk);
QASR_NEIGHBOURS(units, dwoff);
QASR_NEIGHBOURS(drelu, units_inv);
QASR_NEIGHBOURS(row_lanes_log2, row_step);
#undef QASR_NEIGHBOURS
#pragma clang diagnostic pop

// The depthwise half's parameters for tiles of MT <= 2 groups (all but img); false if d is none that it takes.  NA: quads of taps.
bool dw_small_params(const ConvParams& d, int MT, DwParams& p, int& NA);

struct SepChoice { int KCH, MT, NA, NT, KS, splits; bool ragged; };   // KS: wave groups over the pointwise half's input channels

// Can depthwise op d and pointwise op q (q reads d's output and nobody else does) run as one launch?
bool sep_supported(const ConvParams& d, const ConvParams& q);
// ... and with which tile, on 256 units (projection: a pointwise layer of d's input goes along); false if they cannot
bool sep_choice(const ConvParams& d, const ConvParams& q, bool projection, SepChoice& c);
// A depthwise layer's weights as the kernels load them (sep.hip: image)
size_t sep_image_bytes(const ConvParams& d);
hipError_t launch_sep_image(const ConvParams& d, uint32_t* img, hipStream_t st);
// d.x, q.res, q.y set; d.y and q.x are not used
hipError_t launch_sep(const ConvParams& d, const uint32_t* img, const ConvParams& q, hipStream_t st);
// Can the pointwise layer r, which reads d's input and whose output neither d nor q touches, run in the pair's launch?
// Only its geometry, and of its pointers their alignment, are looked at.
bool sep_projection_supported(const ConvParams& d, const ConvParams& q, const ConvParams& r);
hipError_t launch_sep(const ConvParams& d, const uint32_t* img, const ConvParams& q, const ConvParams& r, hipStream_t st);

// one translation unit per tap range (sep_na3.hip ...): the launcher of its instantiations
hipError_t launch_sep_na3(const SepChoice& c, const SepParams& p, size_t lds, hipStream_t st);
hipError_t launch_sep_na4(const SepChoice& c, const SepParams& p, size_t lds, hipStream_t st);
hipError_t launch_sep_na5(const SepChoice& c, const SepParams& p, size_t lds, hipStream_t st);
hipError_t launch_sep_na6(const SepChoice& c, const SepParams& p, size_t lds, hipStream_t st);

}  // namespace qasr
