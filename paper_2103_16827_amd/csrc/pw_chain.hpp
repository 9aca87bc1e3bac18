// Consecutive pointwise layers as one launch: what pw_chain.hip plans and launches.
#pragma once
#include "sep.hpp"

namespace qasr {

constexpr int kMaxChain = 4;         // pointwise layers of a chain

struct ChainLayer {
  const int8_t* w;                   // packed (common.hpp)
  const int32_t *bias, *m, *s;       // bias may be null
  const uint8_t* table;              // of the activation of its output (unary: 256 int8, GLU: 256 16-bit sigmoid codes), or null
  int32_t cin, cout, relu;
  int32_t glu;                       // output channels [0, cout / 2) are values, the rest their gates; only cout / 2 come out
  int32_t glu_m, glu_s;              // rescale of their products
};

struct ChainParams {
  DwParams dw;                       // of the depthwise layer in front; without one only x, xbs, xpitch and Tin are set
  int8_t* y;
  int64_t ybs;
  int32_t ypitch, Tout;
  int32_t xragged, yragged;          // rows not padded to whole aligned 16-byte units
  int32_t n, blocks;                 // layers; 512 x 512 blocks of all of them
  // tiles: the 16-frame groups of a row (batch item) make tpr tiles of g_base groups, the first g_more of them one more
  int32_t tpr, g_base, g_more;
  int32_t wgs, per_xcd;
  int32_t buf[2];                    // LDS: input of the layers of even / odd index
  int32_t const_off, table_off;      // constants of all layers; table of layer l at table_off + 512 l
  int32_t rows_off, row_bytes;       // a wave's scratch of the depthwise layer: rows and its activation's table; then weight rows
  int32_t taps_off;
  float r_tpr;
  ChainLayer layer[kMaxChain];
};

// op[0..n): pointwise layers of which each but the first reads exactly what the one before writes, and nobody else does; table: the
// activation's of its output, or null; glu: that is a GLU's.  dw: the depthwise layer whose output, read by op[0] and nobody else,
// it starts from, or null (its weight image: sep.hpp's).  Whether the pointwise layers can run as one launch, and whether all of them
// can and that is the faster way: only their geometry, and of their pointers the alignment, are looked at.
struct ChainOp {
  ConvParams p;
  const uint8_t* table;
  bool glu;
  int32_t glu_m, glu_s;
};
bool pw_chain_supported(const ChainOp* op, int n);
bool pw_chain_better(const ConvParams* dw, const ChainOp* op, int n);
// dw->x or op[0].p.x and op[n - 1].p.y set; the others' are not used
hipError_t launch_pw_chain(const ConvParams* dw, const uint32_t* img, const ChainOp* op, int n, hipStream_t st);

}  // namespace qasr
