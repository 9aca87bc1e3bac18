// C ABI of the library: argument validation (before any HIP call), kernel dispatch, and the
// encoder executor (a flat op list over activation slots).  See include/qasr.h.
#include "../../include/qasr.h"
#include "kernels.hpp"
#include "pw_chain.hpp"
#include "sep.hpp"
#include "team.hpp"
#include "tuning.hpp"

#include <algorithm>
#include <cmath>
#include <mutex>
#include <new>
#include <vector>

using qasr::ConvParams;

namespace {

thread_local hipError_t g_last_hip = hipSuccess;   // detail behind the last QASR_ERR_HIP

qasr_status hip_status(hipError_t e) {
  if (e == hipSuccess) return QASR_OK;
  g_last_hip = e;
  return QASR_ERR_HIP;
}

constexpr uint32_t kKnownFlags = QASR_FLAG_RELU | QASR_FLAG_W_PACKED;

// Weights have a packed form only for groups == 1 with Cin a multiple of 64 (the matrix-core
// kernels' operand order); otherwise "packed" is the plain order.
bool has_packed_form(const qasr_conv1d_desc* d) { return d->groups == 1 && d->Cin % 64 == 0; }

size_t packed_bytes_of(const qasr_conv1d_desc* d) {
  if (!has_packed_form(d)) return (size_t)((int64_t)d->Cout * (d->groups != 1 ? 1 : d->Cin) * d->k);
  return (size_t)((int64_t)d->k * ((d->Cout + 15) / 16) * 16 * d->Cin);
}

int64_t out_len64(const qasr_conv1d_desc* d) {
  const int64_t span = (int64_t)d->Tin + d->pad_left + d->pad_right - (int64_t)d->dilation * (d->k - 1) - 1;
  return span < 0 ? 0 : span / d->stride + 1;
}

qasr_status check_desc(const qasr_conv1d_desc* d) {
  if (!d) return QASR_ERR_NULL;
  if (d->B < 1 || d->Cin < 1 || d->Cout < 1 || d->Tin < 1 || d->k < 1 || d->stride < 1 ||
      d->dilation < 1 || d->pad_left < 0 || d->pad_right < 0)
    return QASR_ERR_SHAPE;
  if (d->flags & ~kKnownFlags) return QASR_ERR_PARAM;
  if (d->groups != 1 && !(d->groups == d->Cin && d->Cin == d->Cout)) return QASR_ERR_UNSUPPORTED;
  const int64_t Tout = out_len64(d);
  if (Tout < 1 || Tout > 0x7fffffffLL) return QASR_ERR_SHAPE;
  if (d->x_batch_stride < 0 || d->y_batch_stride < 0) return QASR_ERR_SHAPE;
  if (d->x_batch_stride && d->x_batch_stride < (int64_t)d->Cin * d->Tin) return QASR_ERR_SHAPE;
  if (d->y_batch_stride && d->y_batch_stride < (int64_t)d->Cout * Tout) return QASR_ERR_SHAPE;
  return QASR_OK;
}

bool overlaps(const void* a, int64_t na, const void* b, int64_t nb) {
  const uintptr_t a0 = (uintptr_t)a, b0 = (uintptr_t)b;
  return a0 < b0 + (uint64_t)nb && b0 < a0 + (uint64_t)na;
}

ConvParams make_params(const qasr_conv1d_desc* d, const int8_t* x, const int8_t* w, const int32_t* bias,
                       const int32_t* m, const int32_t* s, const int8_t* res, int8_t* y) {
  ConvParams p{};
  p.x = x; p.w = w; p.bias = bias; p.m = m; p.s = s; p.res = res; p.y = y;
  p.B = d->B; p.Cin = d->Cin; p.Cout = d->Cout; p.Tin = d->Tin; p.Tout = (int32_t)out_len64(d);
  p.k = d->k; p.stride = d->stride; p.dil = d->dilation; p.pl = d->pad_left;
  p.depthwise = d->groups != 1;
  p.relu = (d->flags & QASR_FLAG_RELU) ? 1 : 0;
  p.w_packed = (has_packed_form(d) && (d->flags & QASR_FLAG_W_PACKED)) ? 1 : 0;
  p.xbs = d->x_batch_stride ? d->x_batch_stride : (int64_t)d->Cin * d->Tin;
  p.ybs = d->y_batch_stride ? d->y_batch_stride : (int64_t)d->Cout * p.Tout;
  return p;
}

enum class Kernel { Generic, DwMfma, DwPipe, GemmMfma, PwTile, PwPipe, PwWide, ConvPipe, ConvFew };

// the family whose shapes a layer has
Kernel family_of(const ConvParams& p) {
  if (p.n_res_more > 0)      // dense-residual layers: the two kernels whose epilogue adds several operands
    return (!p.depthwise && qasr::conv_pipe_supported(p)) ? Kernel::ConvPipe : Kernel::Generic;
  if (p.depthwise) {
    if (qasr::dw_pipe_supported(p)) return Kernel::DwPipe;
    return qasr::dw_mfma_supported(p) ? Kernel::DwMfma : Kernel::Generic;
  }
  if (qasr::pw_pipe_supported(p)) return Kernel::PwPipe;
  if (qasr::pw_tile_supported(p)) return Kernel::PwTile;
  if (qasr::pw_wide_supported(p)) return Kernel::PwWide;
  if (qasr::conv_pipe_supported(p)) return Kernel::ConvPipe;
  if (qasr::gemm_mfma_supported(p)) return Kernel::GemmMfma;
  return Kernel::Generic;
}

// The kernel that runs a layer.  The one place that decides it: the two pointwise families of the benchmark's
// widths hand launches of some sizes to pw_wide, dense layers of few frames go to conv_few.  It depends on
// lengths, row pitches and pointers (their alignment), not on act_lut, so a layer may get another kernel in
// another call (a float forward gives the ends of an encoder padded rows); whoever asks goes by the answer for
// the call at hand, also for the activation.  split: there is room for the partial sums of a split contraction.
struct Choice {
  Kernel k = Kernel::Generic;
  qasr::FewTile few{};         // ConvFew's
};
Choice choose(const ConvParams& p, bool split) {
  Choice c;
  c.k = family_of(p);
  if (c.k == Kernel::PwTile && qasr::pw_wide_better(p, false)) c.k = Kernel::PwWide;
  else if (c.k == Kernel::PwPipe && qasr::pw_wide_better(p, true)) c.k = Kernel::PwWide;
  else if (c.k == Kernel::ConvPipe && qasr::conv_few_better(p, split, c.few)) c.k = Kernel::ConvFew;
  return c;
}
Choice choose(const ConvParams& p) { return choose(p, p.part != nullptr); }

// kernels whose epilogue applies a unary activation's table (ConvParams::act_lut)
bool applies_act_table(Kernel k) { return k == Kernel::PwPipe || k == Kernel::PwWide || k == Kernel::DwPipe; }

// the kernel's own name, and the name of the family it is counted to
const char* kernel_name(Kernel k) {
  switch (k) {
    case Kernel::DwMfma: return "dw_mfma";
    case Kernel::DwPipe: return "dw_pipe";
    case Kernel::PwTile: return "pw_tile";
    case Kernel::PwPipe: return "pw_pipe";
    case Kernel::PwWide: return "pw_wide";
    case Kernel::GemmMfma: return "gemm_mfma";
    case Kernel::ConvPipe: return "conv_pipe";
    case Kernel::ConvFew: return "conv_few";
    default: return "conv_generic";
  }
}
const char* family_name(Kernel k) {
  return kernel_name(k == Kernel::PwWide ? Kernel::GemmMfma : k == Kernel::ConvFew ? Kernel::ConvPipe : k);
}

// next: a layer that ConvFew runs later, as next_choice says (or null)
qasr_status launch_with(const Choice& c, const ConvParams& p, hipStream_t st, const ConvParams* next = nullptr, const Choice& next_choice = Choice()) {
  hipError_t e;
  switch (c.k) {
    case Kernel::DwMfma: e = qasr::launch_dw_mfma(p, st); break;
    case Kernel::DwPipe: e = qasr::launch_dw_pipe(p, st); break;
    case Kernel::GemmMfma: e = qasr::launch_gemm_mfma(p, st); break;
    case Kernel::PwTile: e = qasr::launch_pw_tile(p, st); break;
    case Kernel::PwPipe: e = qasr::launch_pw_pipe(p, st); break;
    case Kernel::PwWide: e = qasr::launch_pw_wide(p, st); break;
    case Kernel::ConvPipe: e = qasr::launch_conv_pipe(p, st); break;
    case Kernel::ConvFew: e = qasr::launch_conv_few(p, c.few, next, next_choice.few, st); break;
    default: e = qasr::launch_conv_generic(p, st); break;
  }
  return hip_status(e);
}

qasr_status launch(const ConvParams& p, hipStream_t st) { return launch_with(choose(p), p, st); }

// frames between rows of an encoder's own tensors: the row length rounded up to 16
int32_t row_pad(int32_t T) { return (16 - T % 16) % 16; }

size_t round256(size_t n) { return (n + 255) & ~(size_t)255; }

// the library's static device array (qasr_encoder_forward_static)
#define QASR_STATIC_WORKSPACE_BYTES ((size_t)32 << 20)

}  // namespace

struct qasr_encoder {
  struct Op {
    qasr_conv1d_desc d;
    ConvParams p;          // pointers to weights/constants filled in; x / res / y set per forward
    int32_t in_slot, res_slot, out_slot;
    Kernel family;         // for 16-byte aligned, dense input and output
    int32_t n_more_res = 0;
    int32_t more_res_slots[QASR_MAX_RESIDUALS - 1];
    bool has_act = false;
    bool act_fused = false;   // the layer's own kernel applies it (for 16-byte aligned, dense input and output)
    qasr::ActParams act;   // applied in place to the output when has_act
    const uint8_t* act_table = nullptr;   // unary activations: one int8 output per int8 code (kernels with applies_act_table)
    const uint8_t* glu_table = nullptr;   // a GLU's 256 sigmoid codes of 16 bits (chains)
    // This depthwise op and the pointwise op after it may run as one launch (sep.hpp): nothing else reads
    // what it writes.  Its weight image.
    bool sep = false;
    const uint32_t* sep_img = nullptr;
    // This pointwise op (a block's residual projection) and the pair after it read the same tensor and touch none of
    // each other's: the three may run as one launch.
    bool sep_proj = false;
    // This and the next multi - 1 ops are pointwise layers of equal output shape that touch none of each other's
    // outputs (the projections of a dense-residual block): they may run as one launch.  At the first of them; else 0.
    int32_t multi = 0;
    // This and the next chain - 1 ops are pointwise layers of which each but the first reads what the one before writes, and
    // nobody else does: they may run as one launch.  At every op that such a run can begin with; at a depthwise op, whose pair
    // begins one, the number of pointwise layers after it; else 0.
    int32_t chain = 0;
    int32_t in_channels = 0;  // channels of the slot read (p.Cin, or more for a channel-prefix view)
  };
  std::vector<Op> ops;
  std::vector<size_t> slot_off;   // byte offset of slot i in the workspace (slot 0 unused)
  size_t ws_bytes = 0;            // activation buffers, then (from split_off on) what split contractions need
  size_t split_off = 0;
  int64_t in_rows = 0, out_rows = 0;    // rows (batch items x channels) of the network input and output
  int32_t in_T = 0, out_T = 0;          // and their lengths
  bool pitched = false;                 // the slots' rows have a pitch of their own (see rows_of)
  // The same layers over dense rows, for qasr_encoder_forward_static: only where the pitched slots do not
  // fit the static array and the dense ones do (else null).
  qasr_encoder* dense = nullptr;
  int8_t* packed = nullptr;       // device: packed weights of all groups == 1 layers
  // Runs of consecutive ops that one launch of the persistent team kernel executes (team.hip); the
  // ops outside them are launched one by one.
  struct TeamRun {
    int32_t first = 0, count = 0;
    qasr::TeamOp* ops_dev = nullptr;
    qasr::TeamCtl* ctl = nullptr;
  };
  std::vector<TeamRun> runs;
  std::vector<int32_t> run_of;    // per op: index into runs, or -1
  uint32_t* sep_images = nullptr; // device: weight images of the depthwise ops with `sep`
  int8_t* toeplitz = nullptr;     // device: Toeplitz operand images of the depthwise layers inside runs
  int32_t team_wgs = 0;           // workgroups of a team launch (one per compute unit)
};


// ---- team runs: which ops one launch of the persistent kernel takes (host logic only until the
// device arrays are filled).  A run is a maximal stretch of consecutive ops whose shapes the team
// kernel's layer bodies take; it needs at least 8 utterances (one per XCD) and 3 ops to pay.
constexpr int32_t kMinRunOps = 3;

static bool team_record(const qasr_encoder::Op& op, qasr::TeamOp& t) {
  if (op.has_act || op.n_more_res > 0) return false;
  t = qasr::TeamOp{};
  const ConvParams& p = op.p;
  if (p.depthwise) {
    if (!qasr::team_dw_geometry(p, t)) return false;
    t.kind = 1;
  } else {
    if (!qasr::team_pw_geometry(p, t)) return false;
    t.kind = 0;
  }
  t.xbs = p.xbs; t.ybs = p.ybs;
  t.Cin = p.Cin; t.Cout = p.Cout; t.T = p.Tin;
  t.relu = p.relu;
  t.w = p.w; t.bias = p.bias; t.m = p.m; t.s = p.s;
  return true;
}

static qasr_status plan_team_runs(qasr_encoder* e, int32_t n_slots) {
  const int32_t n = (int32_t)e->ops.size();
  e->run_of.assign(n, -1);
  if (!qasr::tuning().team || e->pitched || n < kMinRunOps || e->ops[0].d.B < 8 || n > qasr::kTeamMaxStamps - 2) return QASR_OK;
  std::vector<qasr::TeamOp> rec(n);
  std::vector<char> can(n, 0);
  bool any = false;
  for (int32_t i = 0; i < n; ++i) {
    can[i] = team_record(e->ops[i], rec[i]) ? 1 : 0;
    any = any || can[i];
  }
  if (!any) return QASR_OK;
  e->team_wgs = qasr::team_workgroups();        // (first HIP call of the planner)
  if (e->team_wgs <= 0) return QASR_OK;

  // runs, Toeplitz images
  size_t toep_bytes = 0;
  for (int32_t i = 0; i < n;) {
    if (!can[i]) { ++i; continue; }
    int32_t j = i;
    while (j < n && can[j]) ++j;
    if (j - i >= kMinRunOps) {
      qasr_encoder::TeamRun r;
      r.first = i;
      r.count = j - i;
      for (int32_t q = i; q < j; ++q) {
        e->run_of[q] = (int32_t)e->runs.size();
        if (rec[q].kind == 1) toep_bytes += round256(qasr::team_toeplitz_bytes(rec[q], rec[q].Cout));
      }
      e->runs.push_back(r);
    }
    i = j;
  }
  if (e->runs.empty()) return QASR_OK;
  if (toep_bytes) {
    const hipError_t me = hipMalloc((void**)&e->toeplitz, toep_bytes);
    if (me != hipSuccess) return hip_status(me);
  }
  size_t toff = 0;
  for (qasr_encoder::TeamRun& r : e->runs) {
    // a barrier goes before an op that touches what an op since the last barrier wrote, or writes
    // what one of them read (the first op of a run follows a kernel boundary)
    std::vector<char> written(n_slots, 0), read(n_slots, 0);
    for (int32_t q = r.first; q < r.first + r.count; ++q) {
      const qasr_encoder::Op& op = e->ops[q];
      qasr::TeamOp& t = rec[q];
      const bool hazard = written[op.in_slot] || (op.res_slot >= 0 && written[op.res_slot]) ||
                          written[op.out_slot] || read[op.out_slot];
      t.sync_before = hazard ? 1 : 0;
      if (hazard) {
        std::fill(written.begin(), written.end(), 0);
        std::fill(read.begin(), read.end(), 0);
      }
      read[op.in_slot] = 1;
      if (op.res_slot >= 0) read[op.res_slot] = 1;
      written[op.out_slot] = 1;
      // operands: slot 0 is the network input, the last op's output the network output
      t.in_kind = op.in_slot == 0 ? 0 : 1;
      t.in_off = op.in_slot == 0 ? 0 : (int64_t)e->slot_off[op.in_slot];
      t.res_kind = op.res_slot < 0 ? -1 : (op.res_slot == 0 ? 0 : 1);
      t.res_off = op.res_slot <= 0 ? 0 : (int64_t)e->slot_off[op.res_slot];
      t.out_kind = (q + 1 == n) ? 2 : 1;
      t.out_off = (q + 1 == n) ? 0 : (int64_t)e->slot_off[op.out_slot];
      if (t.kind == 1) {
        int8_t* img = e->toeplitz + toff;
        toff += round256(qasr::team_toeplitz_bytes(t, t.Cout));
        const hipError_t te = qasr::launch_toeplitz_image(op.p.w, op.p.Cout, op.p.k, op.p.dil, t, img, nullptr);
        if (te != hipSuccess) return hip_status(te);
        t.w = img;
      }
    }
    hipError_t me = hipMalloc((void**)&r.ops_dev, sizeof(qasr::TeamOp) * (size_t)r.count);
    if (me == hipSuccess) me = hipMalloc((void**)&r.ctl, sizeof(qasr::TeamCtl));
    if (me == hipSuccess)
      me = hipMemcpy(r.ops_dev, rec.data() + r.first, sizeof(qasr::TeamOp) * (size_t)r.count, hipMemcpyHostToDevice);
    if (me == hipSuccess) me = hipMemset(r.ctl, 0, sizeof(qasr::TeamCtl));
    if (me != hipSuccess) return hip_status(me);
  }
  return QASR_OK;
}

// Rows of op i as it runs: where a tensor lives decides the pitch of its rows.  The slots inside an
// encoder whose lengths are not all multiples of 16 have rows rounded up to 16 frames (`pitched`);
// the network input and output have xpad / ypad frames between rows (0: the caller's dense tensors).
// Every kernel family then sees 16-byte aligned rows whatever the utterance length: before, one frame
// more or less than a multiple of 4 sent every pointwise and dense layer to the one-thread-per-output
// fallback (QuartzNet-15x5, one utterance of 1237 frames: 15.4 ms).
// A pointwise layer between two tensors of equal pitch is run over the pitch itself: its columns are
// independent, the pad columns are computed and ignored.
static void rows_of(const qasr_encoder* e, size_t i, int32_t xpad, int32_t ypad, ConvParams& p) {
  const qasr_encoder::Op& op = e->ops[i];
  p.xpad = op.in_slot == 0 ? xpad : (e->pitched ? row_pad(p.Tin) : 0);
  p.ypad = i + 1 == e->ops.size() ? ypad : (e->pitched ? row_pad(p.Tout) : 0);
  p.xbs = (int64_t)op.in_channels * (p.Tin + p.xpad);
  p.ybs = (int64_t)p.Cout * (p.Tout + p.ypad);
  if (!p.depthwise && p.k == 1 && p.stride == 1 && p.pl == 0 && p.Tin == p.Tout && p.xpad == p.ypad) {
    p.Tin += p.xpad;
    p.Tout += p.ypad;
    p.xpad = p.ypad = 0;
  }
}

extern "C" {

int32_t qasr_conv1d_out_len(const qasr_conv1d_desc* d) {
  const qasr_status st = check_desc(d);
  if (st != QASR_OK) return (int32_t)st;
  return (int32_t)out_len64(d);
}

const char* qasr_conv1d_kernel_name(const qasr_conv1d_desc* d) {
  if (check_desc(d) != QASR_OK) return nullptr;
  const ConvParams p = make_params(d, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr);
  return family_name(family_of(p));
}

const char* qasr_conv1d_launch_name(const qasr_conv1d_desc* d) {
  if (check_desc(d) != QASR_OK) return nullptr;
  const ConvParams p = make_params(d, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr);
  return kernel_name(choose(p).k);
}

qasr_status qasr_conv1d_int8(const qasr_conv1d_desc* d, const int8_t* x, const int8_t* w,
                             const int32_t* bias, const int32_t* m, const int32_t* s,
                             const int8_t* residual, int8_t* y, void* stream) {
  const qasr_status st = check_desc(d);
  if (st != QASR_OK) return st;
  if (!x || !w || !m || !s || !y) return QASR_ERR_NULL;
  const ConvParams p = make_params(d, x, w, bias, m, s, residual, y);
  const int64_t ny = (int64_t)(p.B - 1) * p.ybs + (int64_t)p.Cout * p.Tout;
  const int64_t nx = (int64_t)(p.B - 1) * p.xbs + (int64_t)p.Cin * p.Tin;
  if (overlaps(y, ny, x, nx) || (residual && overlaps(y, ny, residual, ny))) return QASR_ERR_ALIAS;
  return launch(p, (hipStream_t)stream);
}

qasr_status qasr_conv1d_int8_multi(const qasr_conv1d_desc* d, const int8_t* x, const int8_t* w,
                                   const int32_t* bias, const int32_t* m, const int32_t* s,
                                   const int8_t* const* residuals, int32_t n_res, int8_t* y, void* stream) {
  const qasr_status st = check_desc(d);
  if (st != QASR_OK) return st;
  if (!x || !w || !m || !s || !y) return QASR_ERR_NULL;
  if (n_res < 0 || n_res > QASR_MAX_RESIDUALS) return QASR_ERR_PARAM;
  if (n_res > 0 && !residuals) return QASR_ERR_NULL;
  for (int32_t r = 0; r < n_res; ++r)
    if (!residuals[r]) return QASR_ERR_NULL;
  ConvParams p = make_params(d, x, w, bias, m, s, n_res > 0 ? residuals[0] : nullptr, y);
  p.n_res_more = n_res > 1 ? n_res - 1 : 0;
  for (int32_t r = 1; r < n_res; ++r) p.res_more[r - 1] = residuals[r];
  const int64_t ny = (int64_t)(p.B - 1) * p.ybs + (int64_t)p.Cout * p.Tout;
  const int64_t nx = (int64_t)(p.B - 1) * p.xbs + (int64_t)p.Cin * p.Tin;
  if (overlaps(y, ny, x, nx)) return QASR_ERR_ALIAS;
  for (int32_t r = 0; r < n_res; ++r)
    if (overlaps(y, ny, residuals[r], ny)) return QASR_ERR_ALIAS;
  return launch(p, (hipStream_t)stream);
}

size_t qasr_packed_weight_bytes(const qasr_conv1d_desc* d) {
  if (check_desc(d) != QASR_OK) return 0;
  return packed_bytes_of(d);
}

qasr_status qasr_pack_weights(const qasr_conv1d_desc* d, const int8_t* w, int8_t* w_packed, void* stream) {
  const qasr_status st = check_desc(d);
  if (st != QASR_OK) return st;
  if (!w || !w_packed) return QASR_ERR_NULL;
  const size_t n = packed_bytes_of(d);
  const int64_t n_plain = (int64_t)d->Cout * (d->groups != 1 ? 1 : d->Cin) * d->k;
  if (overlaps(w, n_plain, w_packed, (int64_t)n)) return QASR_ERR_ALIAS;
  hipError_t e;
  if (!has_packed_form(d))   // packed form == plain form
    e = hipMemcpyAsync(w_packed, w, n, hipMemcpyDeviceToDevice, (hipStream_t)stream);
  else
    e = qasr::launch_pack_weights(w, w_packed, d->Cout, d->Cin, d->k, (hipStream_t)stream);
  return hip_status(e);
}

qasr_status qasr_requant(const int32_t* acc, int32_t B, int32_t C, int32_t T, const int32_t* bias,
                         const int32_t* m, const int32_t* s, const int8_t* residual, uint32_t flags,
                         int8_t* y, void* stream) {
  if (!acc || !m || !s || !y) return QASR_ERR_NULL;
  if (B < 1 || C < 1 || T < 1) return QASR_ERR_SHAPE;
  if (flags & ~(uint32_t)QASR_FLAG_RELU) return QASR_ERR_PARAM;
  const int64_t n = (int64_t)B * C * T;
  if (overlaps(y, n, acc, 4 * n) || (residual && overlaps(y, n, residual, n))) return QASR_ERR_ALIAS;
  const hipError_t e = qasr::launch_requant(acc, B, C, T, bias, m, s, residual,
                                            (flags & QASR_FLAG_RELU) ? 1 : 0, y, (hipStream_t)stream);
  return hip_status(e);
}

static qasr_status check_alpha(float alpha) {
  if (!(alpha > 0.0f) || !std::isfinite(alpha)) return QASR_ERR_PARAM;
  return alpha / 127.0f > 0.0f ? QASR_OK : QASR_ERR_PARAM;   // (an alpha so small that the step underflows)
}

qasr_status qasr_quantize(const float* x, size_t n, float alpha, int8_t* q, void* stream) {
  if (check_alpha(alpha) != QASR_OK) return QASR_ERR_PARAM;
  const float S = alpha / 127.0f;
  if (n == 0) return QASR_OK;
  if (!x || !q) return QASR_ERR_NULL;
  if (n > ((size_t)1 << 40)) return QASR_ERR_SHAPE;
  if (overlaps(q, (int64_t)n, x, 4 * (int64_t)n)) return QASR_ERR_ALIAS;
  return hip_status(qasr::launch_quantize(x, n, alpha, S, q, (hipStream_t)stream));
}

qasr_status qasr_dequantize(const int8_t* q, size_t n, float S, float* x, void* stream) {
  if (!std::isfinite(S)) return QASR_ERR_PARAM;
  if (n == 0) return QASR_OK;
  if (!x || !q) return QASR_ERR_NULL;
  if (n > ((size_t)1 << 40)) return QASR_ERR_SHAPE;
  if (overlaps(x, 4 * (int64_t)n, q, (int64_t)n)) return QASR_ERR_ALIAS;
  return hip_status(qasr::launch_dequantize(q, n, S, x, (hipStream_t)stream));
}

qasr_status qasr_probe_copy(const void* src, void* dst, size_t bytes, void* stream) {
  if (bytes == 0) return QASR_OK;
  if (!src || !dst) return QASR_ERR_NULL;
  if (bytes % 16 || (uintptr_t)src % 16 || (uintptr_t)dst % 16) return QASR_ERR_SHAPE;
  if (bytes > ((size_t)1 << 40)) return QASR_ERR_SHAPE;
  if (overlaps(dst, (int64_t)bytes, src, (int64_t)bytes)) return QASR_ERR_ALIAS;
  return hip_status(qasr::launch_probe_copy(src, dst, bytes, (hipStream_t)stream));
}

int32_t qasr_probe_mfma_i8_outputs(void) { return qasr::probe_mfma_workgroups(); }

qasr_status qasr_probe_mfma_i8(int32_t iters, int32_t* out, double* ops, void* stream) {
  if (!out || !ops) return QASR_ERR_NULL;
  if (iters < 1 || iters > (1 << 24)) return QASR_ERR_PARAM;
  *ops = qasr::probe_mfma_ops(iters);
  return hip_status(qasr::launch_probe_mfma(iters, out, (hipStream_t)stream));
}

qasr_status qasr_observe_minmax(const float* x, size_t n, float* minmax, void* stream) {
  if (n == 0) return QASR_OK;
  if (!x || !minmax) return QASR_ERR_NULL;
  if (n > ((size_t)1 << 40)) return QASR_ERR_SHAPE;
  if (overlaps(minmax, 8, x, 4 * (int64_t)n)) return QASR_ERR_ALIAS;
  return hip_status(qasr::launch_minmax(x, n, minmax, (hipStream_t)stream));
}

qasr_status qasr_dyadic_from_scale(double M, int32_t* m, int32_t* s) {
  if (!m || !s) return QASR_ERR_NULL;
  int32_t mm, ss;
  if (!qasr::dyadic_from_scale(M, mm, ss)) return QASR_ERR_PARAM;
  *m = mm;
  *s = ss;
  return QASR_OK;
}

qasr_status qasr_fold_bn_quantize(const float* w, const float* conv_bias, const float* gamma, const float* beta,
                                  const float* mean, const float* var, float eps, int32_t Cout, int64_t per_channel,
                                  float S_x, float S_y, int8_t* q_w, int32_t* bias_q, int32_t* m, int32_t* s,
                                  float* S_w, int32_t* bad_count, void* stream) {
  if (!w || !gamma || !beta || !mean || !var || !q_w || !bias_q || !m || !s) return QASR_ERR_NULL;
  if (Cout < 1 || per_channel < 1 || per_channel > ((int64_t)1 << 40) / Cout) return QASR_ERR_SHAPE;
  if (!(S_x > 0.0f) || !std::isfinite(S_x) || !(S_y > 0.0f) || !std::isfinite(S_y) || !(eps >= 0.0f) || !std::isfinite(eps))
    return QASR_ERR_PARAM;
  if (overlaps(q_w, (int64_t)Cout * per_channel, w, 4 * (int64_t)Cout * per_channel)) return QASR_ERR_ALIAS;
  return hip_status(qasr::launch_fold_quantize(w, conv_bias, gamma, beta, mean, var, eps, Cout, per_channel, S_x, S_y, q_w,
                                               bias_q, m, s, S_w, bad_count, (hipStream_t)stream));
}

static qasr_status check_iexp(const qasr_iexp* c) {
  if (!c) return QASR_ERR_NULL;
  if (c->u < 0 || c->u > 16 || c->q_ln2 < 1 || c->q_b < 0 || c->q_b >= ((int64_t)1 << 24) || c->q_c < 0 ||
      c->q_c >= ((int64_t)1 << 48))
    return QASR_ERR_PARAM;
  return QASR_OK;
}

static qasr_status check_act(const qasr_act* a) {
  if (!a) return QASR_ERR_NULL;
  if (a->kind != QASR_ACT_SIGMOID && a->kind != QASR_ACT_SWISH && a->kind != QASR_ACT_GLU) return QASR_ERR_PARAM;
  if (a->m < 0 || a->s < 1 || a->s > 62) return QASR_ERR_PARAM;
  return check_iexp(&a->e);
}

static qasr::ActParams act_params(int32_t kind, int32_t m, int32_t s, const qasr_iexp& e) {
  qasr::ActParams p;
  p.kind = kind; p.m = m; p.s = s; p.u = e.u;
  p.q_ln2 = e.q_ln2; p.q_b = e.q_b; p.q_c = e.q_c;
  return p;
}

qasr_status qasr_iexp_init(double S, int32_t u, qasr_iexp* c) {
  if (!c) return QASR_ERR_NULL;
  if (!(S > 0.0) || !std::isfinite(S) || u < 0 || u > 16) return QASR_ERR_PARAM;
  const double step = std::ldexp(S, -u);                   // S / 2^u, exact
  const double ln2 = 0.6931471805599453;                    // nearest double to ln 2
  const double q_ln2 = std::floor(ln2 / step);
  const double q_b = std::floor(1.353 / step);
  const double q_c = std::floor(0.344 / (0.3585 * step * step));
  if (!(q_ln2 >= 1.0) || !(q_b < 16777216.0)) return QASR_ERR_PARAM;
  c->u = u;
  c->reserved = 0;
  c->q_ln2 = (int64_t)q_ln2;
  c->q_b = (int64_t)q_b;
  c->q_c = (int64_t)q_c;
  return QASR_OK;
}

qasr_status qasr_act_int8(const qasr_act* a, const int8_t* x, int32_t B, int32_t C, int32_t T,
                          int64_t x_batch_stride, int64_t y_batch_stride, int8_t* y, void* stream) {
  const qasr_status st = check_act(a);
  if (st != QASR_OK) return st;
  if (!x || !y) return QASR_ERR_NULL;
  if (B < 1 || B > 65535 || C < 1 || T < 1) return QASR_ERR_SHAPE;
  const int64_t n = (int64_t)C * T, nx = a->kind == QASR_ACT_GLU ? 2 * n : n;
  const int64_t xbs = x_batch_stride ? x_batch_stride : nx, ybs = y_batch_stride ? y_batch_stride : n;
  if (xbs < nx || ybs < n) return QASR_ERR_SHAPE;
  const bool in_place = (const int8_t*)y == x && xbs == ybs;
  if (!in_place && overlaps(y, (int64_t)(B - 1) * ybs + n, x, (int64_t)(B - 1) * xbs + nx)) return QASR_ERR_ALIAS;
  return hip_status(qasr::launch_act(act_params(a->kind, a->m, a->s, a->e), x, y, B, n, xbs, ybs, (hipStream_t)stream));
}

qasr_status qasr_softmax_int32(const qasr_iexp* e, const int32_t* x, int64_t rows, int32_t L, int8_t* y,
                               void* stream) {
  const qasr_status st = check_iexp(e);
  if (st != QASR_OK) return st;
  if (!x || !y) return QASR_ERR_NULL;
  if (rows < 1 || L < 1 || L > 16384 || rows > ((int64_t)1 << 40) / L) return QASR_ERR_SHAPE;
  // the row sum of exponentials (each at most q_b^2 + q_c) times 2^8 must stay inside 64 bits
  if ((double)L * ((double)e->q_b * (double)e->q_b + (double)e->q_c) >= 36028797018963968.0) return QASR_ERR_PARAM;
  if (overlaps(y, rows * L, x, 4 * rows * L)) return QASR_ERR_ALIAS;
  return hip_status(qasr::launch_softmax(act_params(0, 0, 1, *e), x, rows, L, y, (hipStream_t)stream));
}

// ---- buffers for the activation slots.  The caller's slot numbers say which op reads what; which
// memory a value lives in is the library's choice.  It matters: a kernel that writes a buffer which
// the kernel right before it READ runs 3-4 us longer (measured on single layers and on the whole
// encoder: the lines are still held by the L2s of the XCDs that read them, under another
// workgroup-to-XCD mapping, and every write has to displace them), and the two-slot ping-pong of a
// plain layer chain does exactly that in every layer.  So the values are renamed onto physical
// buffers: the output of op i takes the buffer that has been free longest among those that none of
// the `depth` ops before it touched, a new one if there is none (depth + 2 buffers for a plain
// chain).  depth 0 keeps the caller's slots as the buffers.
struct SlotPlan {
  std::vector<int32_t> in, res, out;                 // physical buffer per op (0 = the network input)
  std::vector<std::vector<int32_t>> more;
  std::vector<size_t> bytes;                         // per physical buffer (index 0 unused)
};

struct SlotWire {                                    // what one op reads and writes, in the caller's slots
  int32_t in, res, out;
  std::vector<int32_t> more;
  size_t bytes;                                      // of the value it writes (0: goes to the caller's output)
};

static void plan_slots(const std::vector<SlotWire>& ops, int32_t n_slots, int depth, SlotPlan& pl) {
  const int32_t n_ops = (int32_t)ops.size();
  pl.in.resize(n_ops); pl.res.assign(n_ops, -1); pl.out.resize(n_ops); pl.more.assign(n_ops, {});
  if (depth <= 0) {
    pl.bytes.assign(n_slots, 0);
    for (int32_t i = 0; i < n_ops; ++i) {
      pl.in[i] = ops[i].in; pl.res[i] = ops[i].res; pl.out[i] = ops[i].out;
      pl.more[i] = ops[i].more;
      if (ops[i].bytes > pl.bytes[ops[i].out]) pl.bytes[ops[i].out] = ops[i].bytes;
    }
    return;
  }
  // values: 0 is the network input, i + 1 what op i writes
  std::vector<int32_t> cur(n_slots, -1), last_use(n_ops + 1, -1);
  cur[0] = 0;
  std::vector<std::vector<int32_t>> reads(n_ops);
  for (int32_t i = 0; i < n_ops; ++i) {
    const SlotWire& o = ops[i];
    reads[i].push_back(cur[o.in]);
    if (o.res >= 0) reads[i].push_back(cur[o.res]);
    for (int32_t sl : o.more) reads[i].push_back(cur[sl]);
    for (int32_t v : reads[i]) last_use[v] = i;
    cur[o.out] = i + 1;
  }
  std::vector<int32_t> buf_of(n_ops + 1, -1), holders, free_q;
  buf_of[0] = 0;
  pl.bytes.assign(1, 0);
  std::vector<std::vector<int32_t>> touched(n_ops);
  for (int32_t i = 0; i < n_ops; ++i) {
    for (size_t h = 0; h < holders.size();) {              // values nobody reads from op i on
      if (last_use[holders[h]] < i) {
        free_q.push_back(buf_of[holders[h]]);
        holders.erase(holders.begin() + (long)h);
      } else {
        ++h;
      }
    }
    auto recent = [&](int32_t b) {
      for (int32_t j = i - 1; j >= 0 && j >= i - depth; --j)
        for (int32_t t : touched[j])
          if (t == b) return true;
      return false;
    };
    int32_t b = -1;
    for (size_t q = 0; q < free_q.size(); ++q)
      if (!recent(free_q[q])) {
        b = free_q[q];
        free_q.erase(free_q.begin() + (long)q);
        break;
      }
    if (b < 0) {
      b = (int32_t)pl.bytes.size();
      pl.bytes.push_back(0);
    }
    buf_of[i + 1] = b;
    pl.out[i] = b;
    holders.push_back(i + 1);
    if (ops[i].bytes > pl.bytes[b]) pl.bytes[b] = ops[i].bytes;
    size_t k = 0;
    pl.in[i] = buf_of[reads[i][k++]];
    if (ops[i].res >= 0) pl.res[i] = buf_of[reads[i][k++]];
    for (; k < reads[i].size(); ++k) pl.more[i].push_back(buf_of[reads[i][k]]);
    touched[i].push_back(b);
    for (int32_t v : reads[i]) touched[i].push_back(buf_of[v]);
  }
}

qasr_status qasr_plan_slot_buffers(const int32_t* in_slot, const int32_t* res_slot, const int32_t* out_slot,
                                   int32_t n_ops, int32_t n_slots, int32_t depth, int32_t* in_buf,
                                   int32_t* res_buf, int32_t* out_buf, int32_t* n_buffers) {
  if (!in_slot || !res_slot || !out_slot || !in_buf || !res_buf || !out_buf || !n_buffers) return QASR_ERR_NULL;
  if (n_ops < 1 || n_slots < 2) return QASR_ERR_SHAPE;
  if (depth < 0 || depth > 16) return QASR_ERR_PARAM;
  std::vector<char> live(n_slots, 0);
  live[0] = 1;
  std::vector<SlotWire> w(n_ops);
  for (int32_t i = 0; i < n_ops; ++i) {
    if (in_slot[i] < 0 || in_slot[i] >= n_slots || out_slot[i] < 1 || out_slot[i] >= n_slots || res_slot[i] < -1 ||
        res_slot[i] >= n_slots || out_slot[i] == in_slot[i] || out_slot[i] == res_slot[i])
      return QASR_ERR_PARAM;
    if (!live[in_slot[i]] || (res_slot[i] >= 0 && !live[res_slot[i]])) return QASR_ERR_PARAM;
    live[out_slot[i]] = 1;
    w[i] = SlotWire{in_slot[i], res_slot[i], out_slot[i], {}, (size_t)1};
  }
  SlotPlan pl;
  plan_slots(w, n_slots, depth, pl);
  for (int32_t i = 0; i < n_ops; ++i) { in_buf[i] = pl.in[i]; res_buf[i] = pl.res[i]; out_buf[i] = pl.out[i]; }
  *n_buffers = (int32_t)pl.bytes.size();
  return QASR_OK;
}

// op as part of a chain (its tensors and rows are the caller's business)
static void chain_op(const qasr_encoder::Op& op, qasr::ChainOp& c) {
  c.p = op.p;
  c.glu = op.glu_table != nullptr;
  c.table = c.glu ? op.glu_table : op.act_table;
  c.glu_m = c.glu ? op.act.m : 0;
  c.glu_s = c.glu ? op.act.s : 1;
}

// may_pitch: rows may get a pitch of their own
static qasr_status create_encoder(const qasr_op* ops, int32_t n_ops, int32_t n_slots, bool may_pitch, qasr_encoder** out) {
  if (!ops || !out) return QASR_ERR_NULL;
  if (n_ops < 1 || n_slots < 2) return QASR_ERR_SHAPE;
  *out = nullptr;

  // ---- validation: host only, no HIP call yet
  struct SlotState { bool live = false; int32_t C = 0, T = 0; };
  std::vector<SlotState> slot(n_slots);
  size_t packed_bytes = 0;
  // rows with a pitch of their own: wanted when some length is not a multiple of 16, and possible
  // unless a residual operand would then have another pitch than the output it is added to
  bool ragged = false, pitchable = true;
  for (int32_t i = 0; i < n_ops; ++i) {
    const qasr_op& o = ops[i];
    const qasr_status st = check_desc(&o.d);
    if (st != QASR_OK) return st;
    if (!o.w || !o.m || !o.s) return QASR_ERR_NULL;
    if (o.d.flags & QASR_FLAG_W_PACKED) return QASR_ERR_PARAM;
    if (o.d.y_batch_stride != 0) return QASR_ERR_PARAM;
    if (o.d.B != ops[0].d.B) return QASR_ERR_SHAPE;
    if (o.in_slot < 0 || o.in_slot >= n_slots || o.out_slot < 1 || o.out_slot >= n_slots ||
        o.res_slot < -1 || o.res_slot >= n_slots)
      return QASR_ERR_PARAM;
    if (o.out_slot == o.in_slot || o.out_slot == o.res_slot) return QASR_ERR_PARAM;
    if (o.n_more_res < 0 || o.n_more_res > QASR_MAX_RESIDUALS - 1 || (o.n_more_res > 0 && o.res_slot < 0))
      return QASR_ERR_PARAM;
    for (int32_t r = 0; r < o.n_more_res; ++r) {
      const int32_t sl = o.more_res_slots[r];
      if (sl < 0 || sl >= n_slots || sl == o.out_slot) return QASR_ERR_PARAM;
    }
    if (o.act) {
      const qasr_status as = check_act(o.act);
      if (as != QASR_OK) return as;
      if (o.act->kind == QASR_ACT_GLU && (o.d.Cout & 1)) return QASR_ERR_SHAPE;
      if (o.d.B > 65535) return QASR_ERR_SHAPE;
    }
    if (i == 0) {
      if (ops[0].in_slot != 0) return QASR_ERR_PARAM;
      slot[0].live = true;
      slot[0].T = o.d.Tin;
      slot[0].C = o.d.x_batch_stride ? (int32_t)(o.d.x_batch_stride / o.d.Tin) : o.d.Cin;
    }
    const SlotState& in = slot[o.in_slot];
    if (!in.live || in.T != o.d.Tin) return QASR_ERR_PARAM;
    if (o.d.x_batch_stride == 0 ? in.C != o.d.Cin
                                : (o.d.x_batch_stride != (int64_t)in.C * in.T || o.d.Cin > in.C))
      return QASR_ERR_PARAM;
    const int32_t Tout = (int32_t)out_len64(&o.d);
    if (o.res_slot >= 0) {
      const SlotState& r = slot[o.res_slot];
      if (!r.live || r.C != o.d.Cout || r.T != Tout) return QASR_ERR_PARAM;
    }
    for (int32_t q = 0; q < o.n_more_res; ++q) {
      const SlotState& r = slot[o.more_res_slots[q]];
      if (!r.live || r.C != o.d.Cout || r.T != Tout) return QASR_ERR_PARAM;
    }
    ragged = ragged || row_pad(o.d.Tin) || row_pad(Tout);
    if (row_pad(Tout) && o.res_slot >= 0) {
      if (i + 1 == n_ops || o.res_slot == 0) pitchable = false;
      for (int32_t q = 0; q < o.n_more_res; ++q) pitchable = pitchable && o.more_res_slots[q] != 0;
    }
    if (o.d.Tin < 4 || Tout < 4) pitchable = false;
    slot[o.out_slot].live = true;
    slot[o.out_slot].C = o.d.Cout;
    slot[o.out_slot].T = Tout;
    if (has_packed_form(&o.d)) packed_bytes += round256(packed_bytes_of(&o.d));
    if (o.act) packed_bytes += o.act->kind != QASR_ACT_GLU ? 256 : 512;   // room for a fused activation's table
  }

  qasr_encoder* e = new (std::nothrow) qasr_encoder();
  if (!e) return QASR_ERR_HIP;
  e->pitched = may_pitch && ragged && pitchable;
  // The buffers of the slots with rows of either kind; their bytes in all.
  // They should stay inside the 256 MB memory-side cache together: the deepest plan up to
  // the configured depth whose buffers take at most three quarters of it (QuartzNet-15x5 shape:
  // depth 4 at batch 32, 118 MB; depth 2 at batch 64, 2.44 against 2.46 ms with depth 4 and 2.60
  // with the slots as buffers; at batch 128 even those take 264 MB and every further buffer
  // costs: 4.78 ms with depth 0, 4.92 with 1, 5.53 with 4).
  auto plan_buffers = [&](bool pitched, SlotPlan& pl) {
    std::vector<SlotWire> wires(n_ops);
    for (int32_t i = 0; i < n_ops; ++i) {
      const qasr_op& o = ops[i];
      const int64_t T = out_len64(&o.d);
      wires[i] = SlotWire{o.in_slot, o.res_slot, o.out_slot,
                          std::vector<int32_t>(o.more_res_slots, o.more_res_slots + o.n_more_res),
                          i + 1 == n_ops ? (size_t)0   // (the last op writes the caller's output)
                                         : (size_t)o.d.B * o.d.Cout * (size_t)(T + (pitched ? row_pad((int32_t)T) : 0))};
    }
    const size_t budget = (size_t)192 << 20;
    size_t total = 0;
    for (int depth = qasr::tuning().slot_depth; depth >= 0; --depth) {
      plan_slots(wires, n_slots, depth, pl);
      total = 0;
      for (size_t b = 1; b < pl.bytes.size(); ++b) total += round256(pl.bytes[b]);
      if (total <= budget) break;
    }
    return total;
  };
  SlotPlan plan;
  const size_t plan_bytes = plan_buffers(e->pitched, plan);
  if (e->pitched && plan_bytes > QASR_STATIC_WORKSPACE_BYTES) {
    SlotPlan dense_plan;
    if (plan_buffers(false, dense_plan) <= QASR_STATIC_WORKSPACE_BYTES) {
      const qasr_status ds = create_encoder(ops, n_ops, n_slots, false, &e->dense);
      if (ds != QASR_OK) {
        delete e;
        return ds;
      }
    }
  }
  const int32_t n_bufs = (int32_t)plan.bytes.size();
  e->slot_off.assign(n_bufs, 0);
  size_t off = 0;
  for (int32_t sidx = 1; sidx < n_bufs; ++sidx) {
    e->slot_off[sidx] = off;
    off += round256(plan.bytes[sidx]);
  }
  e->in_rows = (int64_t)ops[0].d.B * slot[0].C;
  e->in_T = slot[0].T;
  {
    const qasr_conv1d_desc& ld = ops[n_ops - 1].d;
    e->out_rows = (int64_t)ld.B * ld.Cout;
    e->out_T = (int32_t)out_len64(&ld);
  }
  e->split_off = off;
  e->ws_bytes = off;

  // ---- one-time device work: pack the dense k>1 weights
  if (packed_bytes) {
    const hipError_t me = hipMalloc((void**)&e->packed, packed_bytes);
    if (me != hipSuccess) { qasr_encoder_destroy(e); return hip_status(me); }
  }
  size_t poff = 0, split_bytes = 0;
  e->ops.resize(n_ops);
  for (int32_t i = 0; i < n_ops; ++i) {
    const qasr_op& o = ops[i];
    qasr_encoder::Op& op = e->ops[i];
    op.d = o.d;
    op.in_slot = plan.in[i]; op.res_slot = plan.res[i]; op.out_slot = plan.out[i];   // (buffers, not the caller's slots)
    const int8_t* w = o.w;
    if (has_packed_form(&o.d)) {
      int8_t* wp = e->packed + poff;
      poff += round256(packed_bytes_of(&o.d));
      const hipError_t pe = qasr::launch_pack_weights(o.w, wp, o.d.Cout, o.d.Cin, o.d.k, nullptr);
      if (pe != hipSuccess) {
        qasr_encoder_destroy(e);
        return hip_status(pe);
      }
      w = wp;
      op.d.flags |= QASR_FLAG_W_PACKED;
    }
    op.p = make_params(&op.d, nullptr, w, o.bias, o.m, o.s, nullptr, nullptr);
    op.n_more_res = o.n_more_res;
    op.p.n_res_more = o.n_more_res;
    for (int32_t r = 0; r < o.n_more_res; ++r) op.more_res_slots[r] = plan.more[i][r];
    op.in_channels = (int32_t)(op.p.xbs / op.p.Tin);
    {
      ConvParams rp = op.p;               // (the pointers are unknown yet: the choice for aligned ones)
      rows_of(e, i, 0, 0, rp);
      op.family = family_of(rp);
      op.act_fused = o.act && o.act->kind != QASR_ACT_GLU && applies_act_table(choose(rp).k);
      if (op.family == Kernel::ConvPipe) split_bytes = std::max(split_bytes, qasr::conv_pipe_split_bytes(rp));
    }
    if (o.act) {
      op.has_act = true;
      op.act = act_params(o.act->kind, o.act->m, o.act->s, o.act->e);
      // A unary activation's table (one int8 output per int8 code) is built here once by the activation's
      // own integer arithmetic: the pipelined depthwise, the pipelined and the wide pointwise kernel and the
      // depthwise + pointwise pairs apply it in their epilogue, after any other kernel the activation is a
      // pass of its own.
      if (o.act->kind != QASR_ACT_GLU) {
        uint8_t* const table = reinterpret_cast<uint8_t*>(e->packed + poff);
        poff += 256;
        const hipError_t te = qasr::launch_act_table(op.act, table, nullptr);
        if (te != hipSuccess) {
          qasr_encoder_destroy(e);
          return hip_status(te);
        }
        op.act_table = table;
      } else {
        uint16_t* const table = reinterpret_cast<uint16_t*>(e->packed + poff);
        poff += 512;
        const hipError_t te = qasr::launch_glu_table(op.act, table, nullptr);
        if (te != hipSuccess) {
          qasr_encoder_destroy(e);
          return hip_status(te);
        }
        op.glu_table = reinterpret_cast<const uint8_t*>(table);
      }
    }
  }
  if (split_bytes && e->split_off) e->ws_bytes =   // (an encoder that needs no workspace goes on needing none)
      e->split_off + round256(split_bytes) + round256(4 * qasr::kConvSplitCounters);
  // op i + 1 reads what op i writes, as its input and nothing else, and no other op does
  auto read_by_next_only = [&](int32_t i) {
    const qasr_op &o = ops[i], &q = ops[i + 1];
    if (q.in_slot != o.out_slot || q.res_slot == o.out_slot) return false;
    for (int32_t r = 0; r < q.n_more_res; ++r)
      if (q.more_res_slots[r] == o.out_slot) return false;
    for (int32_t j = i + 2; j < n_ops && ops[j - 1].out_slot != o.out_slot; ++j) {
      if (ops[j].in_slot == o.out_slot || ops[j].res_slot == o.out_slot) return false;
      for (int32_t r = 0; r < ops[j].n_more_res; ++r)
        if (ops[j].more_res_slots[r] == o.out_slot) return false;
    }
    return true;
  };
  // only the first half of op i's channels, a GLU's products, is ever read, and by other ops only
  auto read_by_half = [&](int32_t i) {
    const qasr_op& o = ops[i];
    for (int32_t j = i + 1; j < n_ops; ++j) {
      if (ops[j].in_slot == o.out_slot && 2 * ops[j].d.Cin > o.d.Cout) return false;
      if (ops[j].res_slot == o.out_slot) return false;
      for (int32_t r = 0; r < ops[j].n_more_res; ++r)
        if (ops[j].more_res_slots[r] == o.out_slot) return false;
      if (ops[j].out_slot == o.out_slot) return true;
    }
    return i + 1 < n_ops;
  };
  // ---- depthwise + pointwise pairs that run as one launch
  if (!e->pitched && qasr::tuning().team) {
    // (the experimental team kernel takes such layers one by one)
  } else {
    std::vector<size_t> img_off(n_ops, 0);
    size_t img_bytes = 0;
    for (int32_t i = 0; i + 1 < n_ops; ++i) {
      const qasr_op &o = ops[i], &q = ops[i + 1];
      if (o.d.groups == 1 || q.in_slot != o.out_slot || q.res_slot == o.out_slot || o.out_slot == 0) continue;
      if ((o.act && o.act->kind == QASR_ACT_GLU) || q.act) continue;
      if (e->ops[i + 1].out_slot == e->ops[i].in_slot && i + 2 != n_ops) continue;   // (tiles read their neighbours' input)
      if (!read_by_next_only(i)) continue;
      ConvParams dp = e->ops[i].p, qp = e->ops[i + 1].p;
      rows_of(e, i, row_pad(dp.Tin), row_pad(dp.Tout), dp);
      rows_of(e, i + 1, row_pad(qp.Tin), row_pad(qp.Tout), qp);
      if (!qasr::sep_supported(dp, qp)) continue;
      e->ops[i].sep = true;
      img_off[i] = img_bytes;
      img_bytes += round256(qasr::sep_image_bytes(dp));
    }
    for (int32_t i = 0; i + 2 < n_ops; ++i) {
      const qasr_op &o = ops[i], &d = ops[i + 1];
      if (!e->ops[i + 1].sep || o.act || o.res_slot >= 0 || o.d.groups != 1 || o.in_slot != d.in_slot) continue;
      qasr_encoder::Op &r = e->ops[i], &dw = e->ops[i + 1], &pw = e->ops[i + 2];   // (their slots are buffers)
      r.sep_proj = r.in_channels == dw.in_channels && r.out_slot != dw.in_slot && r.out_slot != pw.out_slot && r.out_slot != pw.res_slot;
    }
    // ---- runs of independent pointwise layers of equal output shape
    for (int32_t i = 0; i + 1 < n_ops;) {
      auto plain = [&](int32_t j) {
        const qasr_op& o = ops[j];
        return o.d.groups == 1 && o.d.k == 1 && o.d.stride == 1 && o.d.pad_left == 0 && o.d.pad_right == 0 && o.res_slot < 0 && !o.act &&
               !e->ops[j].sep_proj && !(j > 0 && e->ops[j - 1].sep);       // (those go out with a pair)
      };
      int32_t n = 0;
      while (i + n < n_ops && n < qasr::kMaxMulti && plain(i + n) && ops[i + n].d.Cout == ops[i].d.Cout &&
             ops[i + n].d.Tin == ops[i].d.Tin) {
        bool apart = true;                    // (slots are buffers by now; the last op of all writes the caller's output)
        for (int32_t j = 0; j < n && apart; ++j)
          apart = e->ops[i + j].out_slot != e->ops[i + n].in_slot && e->ops[i + j].out_slot != e->ops[i + n].out_slot &&
                  e->ops[i + n].out_slot != e->ops[i + j].in_slot;
        if (!apart || i + n + 1 == n_ops) break;
        ++n;
      }
      if (n > 1) e->ops[i].multi = n;
      i += n > 1 ? n : 1;
    }
    // ---- runs of pointwise layers, each the only reader of the one before
    for (int32_t i = 0; i + 1 < n_ops; ++i) {
      auto plain = [&](int32_t j) {
        const qasr_op& o = ops[j];
        return o.d.groups == 1 && o.d.k == 1 && o.d.stride == 1 && o.d.pad_left == 0 && o.d.pad_right == 0 && o.res_slot < 0 &&
               (!o.act || o.act->kind != QASR_ACT_GLU || read_by_half(j));
      };
      int32_t n = 0;
      while (i + n < n_ops && n < qasr::kMaxChain && plain(i + n)) {
        ++n;
        if (i + n == n_ops || !read_by_next_only(i + n - 1)) break;
      }
      for (; n > 1; --n) {                    // (slots are buffers by now; the last op of all writes the caller's output)
        if (i + n < n_ops && e->ops[i + n - 1].out_slot == e->ops[i].in_slot) continue;
        qasr::ChainOp c[qasr::kMaxChain];
        for (int32_t j = 0; j < n; ++j) {
          chain_op(e->ops[i + j], c[j]);
          rows_of(e, i + j, row_pad(c[j].p.Tin), row_pad(c[j].p.Tout), c[j].p);
        }
        if (qasr::pw_chain_supported(c, n)) break;
      }
      e->ops[i].chain = n > 1 ? n : 0;
    }
    for (int32_t i = 0; i + 1 < n_ops; ++i) {  // ... and the depthwise layer before them (whose tiles read their neighbours' input)
      qasr_encoder::Op& op = e->ops[i];
      const int32_t n = op.sep ? e->ops[i + 1].chain : 0;
      if (n < 2 || (i + 1 + n < n_ops && e->ops[i + n].out_slot == op.in_slot)) continue;
      op.chain = n;
    }
    hipError_t he = img_bytes ? hipMalloc((void**)&e->sep_images, img_bytes) : hipSuccess;
    for (int32_t i = 0; i < n_ops && he == hipSuccess; ++i) {
      qasr_encoder::Op& op = e->ops[i];
      if (!op.sep) continue;
      uint32_t* const img = e->sep_images + img_off[i] / 4;
      op.sep_img = img;
      he = qasr::launch_sep_image(op.p, img, nullptr);
    }
    if (he != hipSuccess) {
      qasr_encoder_destroy(e);
      return hip_status(he);
    }
  }
  {
    const qasr_status ts = plan_team_runs(e, n_bufs);
    if (ts != QASR_OK) {
      qasr_encoder_destroy(e);
      return ts;
    }
  }
  if (packed_bytes || e->sep_images || !e->runs.empty()) {
    const hipError_t se = hipStreamSynchronize(nullptr);
    if (se != hipSuccess) {
      qasr_encoder_destroy(e);
      return hip_status(se);
    }
  }
  *out = e;
  return QASR_OK;
}

qasr_status qasr_encoder_create(const qasr_op* ops, int32_t n_ops, int32_t n_slots, qasr_encoder** out) {
  return create_encoder(ops, n_ops, n_slots, true, out);
}

size_t qasr_encoder_workspace_bytes(const qasr_encoder* e) { return e ? e->ws_bytes : 0; }

int32_t qasr_encoder_num_ops(const qasr_encoder* e) { return e ? (int32_t)e->ops.size() : 0; }

const char* qasr_encoder_op_kernel(const qasr_encoder* e, int32_t i) {
  if (!e || i < 0 || i >= (int32_t)e->ops.size()) return nullptr;
  return family_name(e->ops[i].family);
}

// whether a forward's workspace has room for the partial sums of split contractions
static bool has_split_room(const qasr_encoder* e) { return e->ws_bytes > e->split_off; }

// the pair at op i may take the projection r before it along
static bool projection_with_pair(const ConvParams& r, const ConvParams& d, const ConvParams& q) {
  return qasr::sep_supported(d, q) && qasr::sep_projection_supported(d, q, r);
}

// whether op i and op i + 1 run as one launch over 16-byte aligned, dense input and output
static bool runs_as_pair(const qasr_encoder* e, size_t i) {
  if (!e->ops[i].sep) return false;
  ConvParams p = e->ops[i].p, q = e->ops[i + 1].p;
  rows_of(e, i, 0, 0, p);
  rows_of(e, i + 1, 0, 0, q);
  return qasr::sep_supported(p, q);
}

// whether the multi ops from op i on run as one launch
static bool runs_as_multi(const qasr_encoder* e, size_t i) {
  const int32_t n = e->ops[i].multi;
  if (n < 2) return false;
  ConvParams p[qasr::kMaxMulti];
  for (int32_t j = 0; j < n; ++j) {
    p[j] = e->ops[i + j].p;
    rows_of(e, i + j, 0, 0, p[j]);
  }
  return qasr::pw_multi_better(p, n);
}

// the ops that run as one launch, a chain, from op i on (0: none)
static int32_t runs_as_chain(const qasr_encoder* e, size_t i) {
  const int32_t n = e->ops[i].chain, from_dw = e->ops[i].sep ? 1 : 0;
  if (n < 2) return 0;
  qasr::ChainOp c[qasr::kMaxChain];
  for (int32_t j = 0; j < n; ++j) {
    chain_op(e->ops[i + from_dw + j], c[j]);
    rows_of(e, i + from_dw + j, 0, 0, c[j].p);
  }
  ConvParams d = e->ops[i].p;
  rows_of(e, i, 0, 0, d);
  return qasr::pw_chain_better(from_dw ? &d : nullptr, c, n) ? n + from_dw : 0;
}

// the same for op i, a projection, with ops i + 1 and i + 2
static bool runs_with_pair(const qasr_encoder* e, size_t i) {
  if (!e->ops[i].sep_proj) return false;
  ConvParams r = e->ops[i].p, p = e->ops[i + 1].p, q = e->ops[i + 2].p;
  rows_of(e, i, 0, 0, r);
  rows_of(e, i + 1, 0, 0, p);
  rows_of(e, i + 2, 0, 0, q);
  return projection_with_pair(r, p, q);
}

int32_t qasr_encoder_op_launch(const qasr_encoder* e, int32_t i, const char** kernel) {
  if (!e || i < 0 || i >= (int32_t)e->ops.size()) return -1;
  for (int32_t first = 0;;) {                       // launch after launch, as a forward goes
    const char* name = "sep";
    int32_t n = runs_as_chain(e, (size_t)first);
    if (n) name = "pw_chain";
    else if (runs_as_multi(e, (size_t)first)) n = e->ops[first].multi, name = "pw_wide";
    else if (runs_with_pair(e, (size_t)first)) n = 3;
    else if (runs_as_pair(e, (size_t)first)) n = 2;
    else n = 1, name = nullptr;
    if (first + n <= i) {
      first += n;
      continue;
    }
    if (kernel) {
      ConvParams p = e->ops[i].p;
      rows_of(e, (size_t)i, 0, 0, p);
      *kernel = name ? name : kernel_name(choose(p, has_split_room(e)).k);
    }
    return first;
  }
}

int32_t qasr_encoder_op_act_fused(const qasr_encoder* e, int32_t i) {
  if (!e || i < 0 || i >= (int32_t)e->ops.size()) return -1;
  return e->ops[i].act_fused ? 1 : 0;
}

int32_t qasr_encoder_op_in_team(const qasr_encoder* e, int32_t i) {
  if (!e || i < 0 || i >= (int32_t)e->ops.size()) return -1;
  return e->run_of.empty() ? 0 : (e->run_of[i] >= 0 ? 1 : 0);
}

struct ForwardHow {
  int team = 1;                   // 0: no team runs, 1: the planned ones, 2: with the team kernel's clock stamps
  bool pairs = true;              // depthwise + pointwise pairs as one launch
  int32_t xpad = 0, ypad = 0;     // frames between the rows of x and y (pitched encoders only; 0 = the caller's dense tensors)
  bool split = true;              // the workspace has room for the partial sums of split contractions
  // ev[i] is recorded where the launch that begins with op i begins (and began[i] set), ev[n] at the end
  hipEvent_t* ev = nullptr;
  char* began = nullptr;
};

static qasr_status forward_impl(const qasr_encoder* e, const int8_t* x, int8_t* y, void* workspace,
                                size_t workspace_bytes, hipStream_t st, const ForwardHow& how = ForwardHow()) {
  const int32_t xpad = how.xpad, ypad = how.ypad;
  bool split = how.split;
  auto begin = [&](size_t i) {
    if (!how.ev) return hipSuccess;
    how.began[i] = 1;
    return hipEventRecord(how.ev[i], st);
  };
  if (!e || !x || !y) return QASR_ERR_NULL;
  if (e->ws_bytes && (!workspace || ((uintptr_t)workspace & 255) || workspace_bytes < (split ? e->ws_bytes : e->split_off)))
    return QASR_ERR_WORKSPACE;
  int8_t* ws = (int8_t*)workspace;
  const size_t n = e->ops.size();
  // y may lie over x, which is read before the last op begins: such a call gets no launch whose tiles would write y while others of
  // it still read x
  const bool y_over_x = overlaps(x, e->in_rows * (e->in_T + xpad), y, e->out_rows * (e->out_T + ypad));
  auto keeps_apart = [&](size_t first, size_t count) {
    if (!y_over_x || first + count != n) return false;
    for (size_t j = first; j + 1 < n; ++j)
      if (e->ops[j].in_slot == 0 || e->ops[j].res_slot == 0) return true;
    return false;
  };
  // (the team kernel's loads want 16-byte aligned tensors, like the kernels it replaces)
  const bool use_team = how.team && !e->runs.empty() && ((uintptr_t)x % 16 == 0) && ((uintptr_t)y % 16 == 0) && !y_over_x;
  // room for the partial sums of split contractions, and their counters (zero between layers from here on)
  split = split && has_split_room(e);
  const size_t split_bytes = split ? e->ws_bytes - e->split_off - round256(4 * qasr::kConvSplitCounters) : 0;
  if (const hipError_t be = begin(0); be != hipSuccess) return hip_status(be);
  if (split) {
    const hipError_t ce = qasr::launch_conv_split_clear((unsigned*)(ws + e->split_off + split_bytes), st);
    if (ce != hipSuccess) return hip_status(ce);
  }
  // layer i's parameters with this call's tensors
  auto bind = [&](size_t i, ConvParams& p) {
    const qasr_encoder::Op& op = e->ops[i];
    p = op.p;
    rows_of(e, i, xpad, ypad, p);
    if (split) {
      p.part = (int32_t*)(ws + e->split_off);
      p.part_bytes = split_bytes;
      p.part_count = (unsigned*)(ws + e->split_off + split_bytes);
    }
    p.x = op.in_slot == 0 ? x : ws + e->slot_off[op.in_slot];
    p.res = op.res_slot < 0 ? nullptr : (op.res_slot == 0 ? x : ws + e->slot_off[op.res_slot]);
    p.y = (i + 1 == n) ? y : ws + e->slot_off[op.out_slot];
    for (int32_t r = 0; r < op.n_more_res; ++r)
      p.res_more[r] = op.more_res_slots[r] == 0 ? x : ws + e->slot_off[op.more_res_slots[r]];
  };
  Choice chosen;                                    // layer chosen_for's, which the one before has asked for
  size_t chosen_for = n;                            // (n: none)
  for (size_t i = 0; i < n; ++i) {
    if (use_team && e->run_of[i] >= 0) {
      const qasr_encoder::TeamRun& r = e->runs[e->run_of[i]];
      const hipError_t te = qasr::launch_team(r.ops_dev, r.count, x, ws, y, e->ops[0].d.B, r.ctl, e->team_wgs,
                                              how.team == 2 ? 1 : 0, st);
      if (te != hipSuccess) return hip_status(te);
      i = (size_t)(r.first + r.count) - 1;
      continue;
    }
    const qasr_encoder::Op& op = e->ops[i];
    ConvParams p;
    bind(i, p);
    if (i > 0)
      if (const hipError_t be = begin(i); be != hipSuccess) return hip_status(be);
    if (how.pairs) {
      // a chain of pointwise layers, from a depthwise layer on or by itself
      if (const int32_t cn = op.chain; cn > 1) {
        const int32_t from_dw = op.sep ? 1 : 0;
        qasr::ChainOp c[qasr::kMaxChain];
        for (int32_t j = 0; j < cn; ++j) {
          chain_op(e->ops[i + from_dw + j], c[j]);
          bind(i + from_dw + j, c[j].p);
        }
        ConvParams d = p;
        d.act_lut = op.act_table;
        if (!keeps_apart(i, (size_t)(cn + from_dw)) && qasr::pw_chain_better(from_dw ? &d : nullptr, c, cn)) {
          const hipError_t ce = qasr::launch_pw_chain(from_dw ? &d : nullptr, op.sep_img, c, cn, st);
          if (ce != hipSuccess) return hip_status(ce);
          i += (size_t)(cn + from_dw) - 1;
          continue;
        }
      }
    }
    if (op.multi > 1 && how.pairs) {
      ConvParams l[qasr::kMaxMulti];
      l[0] = p;
      for (int32_t j = 1; j < op.multi; ++j) bind(i + j, l[j]);
      if (qasr::pw_multi_better(l, op.multi)) {
        const hipError_t me = qasr::launch_pw_multi(l, op.multi, st);
        if (me != hipSuccess) return hip_status(me);
        i += (size_t)op.multi - 1;
        continue;
      }
    }
    if (op.sep_proj && how.pairs) {
      ConvParams d, q;
      bind(i + 1, d);
      bind(i + 2, q);
      d.act_lut = e->ops[i + 1].act_table;
      if (!keeps_apart(i, 3) && projection_with_pair(p, d, q)) {
        const hipError_t se = qasr::launch_sep(d, e->ops[i + 1].sep_img, q, p, st);
        if (se != hipSuccess) return hip_status(se);
        i += 2;
        continue;
      }
    }
    if (op.sep && how.pairs) {
      ConvParams q;
      bind(i + 1, q);
      p.act_lut = op.act_table;                  // (of the activation between the two)
      if (!keeps_apart(i, 2) && qasr::sep_supported(p, q)) {
        const hipError_t se = qasr::launch_sep(p, op.sep_img, q, st);
        if (se != hipSuccess) return hip_status(se);
        ++i;
        continue;
      }
    }
    // (the kernel of this call decides who applies a unary activation: its epilogue, or a pass of its own)
    const Choice c = chosen_for == i ? chosen : choose(p);
    p.act_lut = applies_act_table(c.k) ? op.act_table : nullptr;
    // (the next layer of conv_few's, pointwise ones between them passed over: their weights leave room in the L2s)
    ConvParams later;
    const ConvParams* next = nullptr;
    if (c.k == Kernel::ConvFew) {
      size_t j = i + 1;
      while (j < n && e->ops[j].p.k < 2) ++j;
      if (j < n) {
        bind(j, later);
        chosen = choose(later);
        chosen_for = j;
        if (chosen.k == Kernel::ConvFew) next = &later;
      }
    }
    const qasr_status s = launch_with(c, p, st, next, chosen);
    if (s != QASR_OK) return s;
    if (op.has_act && !p.act_lut) {
      const bool glu = op.act.kind == QASR_ACT_GLU;
      const int64_t n_out = (int64_t)(glu ? p.Cout / 2 : p.Cout) * (p.Tout + p.ypad);
      const hipError_t ae = qasr::launch_act(op.act, p.y, p.y, p.B, n_out, p.ybs, p.ybs, st);
      if (ae != hipSuccess) return hip_status(ae);
    }
  }
  return hip_status(how.ev ? hipEventRecord(how.ev[n], st) : hipSuccess);
}

qasr_status qasr_encoder_forward(const qasr_encoder* e, const int8_t* x, int8_t* y, void* workspace,
                                 size_t workspace_bytes, void* stream) {
  return forward_impl(e, x, y, workspace, workspace_bytes, (hipStream_t)stream);
}

// ---- the forward for callers that can neither allocate nor pass a workspace: the activation slots
// live in a static device array of the library.  The array's name is only a host-side stand-in; its
// device address is looked up once per device and kept.
static __device__ __align__(256) unsigned char scratch[QASR_STATIC_WORKSPACE_BYTES];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// device address of `scratch` on the current device (looked up at the first call on that device)
qasr_status static_scratch(void** out) {
  int dev = 0;
  const hipError_t ge = hipGetDevice(&dev);
  if (ge != hipSuccess) return hip_status(ge);
  if (dev < 0 || dev >= kMaxDevices) return QASR_ERR_UNSUPPORTED;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    const hipError_t se = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (se != hipSuccess) return hip_status(se);
    if (!ptr || ((uintptr_t)ptr & 255)) return QASR_ERR_WORKSPACE;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return QASR_OK;
}

}  // namespace

size_t qasr_static_workspace_bytes(void) { return QASR_STATIC_WORKSPACE_BYTES; }

qasr_status qasr_encoder_forward_static(const qasr_encoder* e, const int8_t* x, int8_t* y, void* stream) {
  if (!e || !x || !y) return QASR_ERR_NULL;
  if (e->dense) e = e->dense;
  if (e->split_off > QASR_STATIC_WORKSPACE_BYTES) return QASR_ERR_WORKSPACE;    // before any HIP call
  void* ws = nullptr;
  const qasr_status st = static_scratch(&ws);
  if (st != QASR_OK) return st;
  // every slot is written in full by the op that produces it before any op reads it: nothing in the
  // array has to start at zero, whatever an earlier call left there
  ForwardHow how;
  how.split = e->ws_bytes <= QASR_STATIC_WORKSPACE_BYTES;
  return forward_impl(e, x, y, ws, QASR_STATIC_WORKSPACE_BYTES, (hipStream_t)stream, how);
}

qasr_status qasr_encoder_forward_layerwise(const qasr_encoder* e, const int8_t* x, int8_t* y, void* workspace,
                                           size_t workspace_bytes, void* stream) {
  ForwardHow how;
  how.team = 0;
  how.pairs = false;
  return forward_impl(e, x, y, workspace, workspace_bytes, (hipStream_t)stream, how);
}

qasr_status qasr_encoder_team_check(const qasr_encoder* e, int32_t* aborted) {
  if (!e || !aborted) return QASR_ERR_NULL;
  *aborted = 0;
  for (const qasr_encoder::TeamRun& r : e->runs) {
    uint32_t flag = 0;
    const hipError_t ce = hipMemcpy(&flag, &r.ctl->abort, sizeof(flag), hipMemcpyDeviceToHost);
    if (ce != hipSuccess) return hip_status(ce);
    if (flag) *aborted = 1;
  }
  return QASR_OK;
}

qasr_status qasr_encoder_forward_team_stamps(const qasr_encoder* e, const int8_t* x, int8_t* y, void* workspace,
                                             size_t workspace_bytes, void* stream, float* op_us) {
  if (!e || !op_us) return QASR_ERR_NULL;
  const size_t n = e->ops.size();
  for (size_t i = 0; i < n; ++i) op_us[i] = 0.f;
  ForwardHow how;
  how.team = 2;
  qasr_status st = forward_impl(e, x, y, workspace, workspace_bytes, (hipStream_t)stream, how);
  if (st != QASR_OK) return st;
  if (hipStreamSynchronize((hipStream_t)stream) != hipSuccess) return QASR_ERR_HIP;
  std::vector<unsigned long long> stamp(qasr::kTeamMaxStamps);
  for (const qasr_encoder::TeamRun& r : e->runs) {
    const hipError_t ce = hipMemcpy(stamp.data(), r.ctl->stamp, sizeof(unsigned long long) * (size_t)(r.count + 1),
                                    hipMemcpyDeviceToHost);
    if (ce != hipSuccess) return hip_status(ce);
    for (int32_t q = 0; q < r.count; ++q)       // the clock runs at 100 MHz
      op_us[r.first + q] = (float)((double)(stamp[q + 1] - stamp[q]) * 0.01);
  }
  return st;
}

// int8 copies of the network input and output of a float forward, in rows of the slots' pitch
static size_t f32_copy_bytes(const qasr_encoder* e, int64_t rows, int32_t T) {
  return round256((size_t)rows * (T + (e->pitched ? row_pad(T) : 0)));
}

size_t qasr_encoder_workspace_bytes_f32(const qasr_encoder* e) {
  return e ? e->ws_bytes + f32_copy_bytes(e, e->in_rows, e->in_T) + f32_copy_bytes(e, e->out_rows, e->out_T) : 0;
}

qasr_status qasr_encoder_forward_f32(const qasr_encoder* e, const float* x, float alpha, float S_out, float* y,
                                     void* workspace, size_t workspace_bytes, void* stream) {
  if (!e || !x || !y) return QASR_ERR_NULL;
  if (!workspace || ((uintptr_t)workspace & 255) || workspace_bytes < qasr_encoder_workspace_bytes_f32(e))
    return QASR_ERR_WORKSPACE;
  int8_t* xq = (int8_t*)workspace + e->ws_bytes;
  int8_t* yq = xq + f32_copy_bytes(e, e->in_rows, e->in_T);
  const int32_t xpad = e->pitched ? row_pad(e->in_T) : 0, ypad = e->pitched ? row_pad(e->out_T) : 0;
  const hipStream_t st_ = (hipStream_t)stream;
  qasr_status st;
  if (xpad == 0) {
    st = qasr_quantize(x, (size_t)e->in_rows * e->in_T, alpha, xq, stream);
  } else {
    st = check_alpha(alpha);
    if (st == QASR_OK)
      st = hip_status(qasr::launch_quantize_rows(x, e->in_rows, e->in_T, alpha, alpha / 127.0f, xq, e->in_T + xpad, st_));
  }
  if (st == QASR_OK) {
    ForwardHow how;
    how.xpad = xpad;
    how.ypad = ypad;
    st = forward_impl(e, xq, yq, workspace, e->ws_bytes ? e->ws_bytes : workspace_bytes, st_, how);
  }
  if (st != QASR_OK) return st;
  if (ypad == 0) return qasr_dequantize(yq, (size_t)e->out_rows * e->out_T, S_out, y, stream);
  if (!std::isfinite(S_out)) return QASR_ERR_PARAM;
  return hip_status(qasr::launch_dequantize_rows(yq, e->out_rows, e->out_T, e->out_T + ypad, S_out, y, st_));
}

qasr_status qasr_encoder_forward_timed(const qasr_encoder* e, const int8_t* x, int8_t* y, void* workspace,
                                       size_t workspace_bytes, void* stream, float* op_ms) {
  if (!e || !op_ms) return QASR_ERR_NULL;
  const size_t n = e->ops.size();
  std::vector<hipEvent_t> ev(n + 1, nullptr);
  hipEvent_t cal[2] = {nullptr, nullptr};
  qasr_status st = QASR_OK;
  for (size_t i = 0; i <= n && st == QASR_OK; ++i)
    if (hipEventCreate(&ev[i]) != hipSuccess) st = QASR_ERR_HIP;
  for (int i = 0; i < 2 && st == QASR_OK; ++i)
    if (hipEventCreate(&cal[i]) != hipSuccess) st = QASR_ERR_HIP;
  // An event record between two kernels costs device time of its own.  The same forward is run
  // once without inner events (bracketed by two) and once with them; the difference of the two
  // totals, spread evenly over the launches, is taken off every launch's interval, so that the times add
  // up to the duration of the undisturbed forward.
  std::vector<char> began(n + 1, 0);
  ForwardHow plain_how, how;
  plain_how.team = how.team = 0;
  how.ev = ev.data();
  how.began = began.data();
  if (st == QASR_OK && hipEventRecord(cal[0], (hipStream_t)stream) != hipSuccess) st = QASR_ERR_HIP;
  if (st == QASR_OK) st = forward_impl(e, x, y, workspace, workspace_bytes, (hipStream_t)stream, plain_how);
  if (st == QASR_OK && hipEventRecord(cal[1], (hipStream_t)stream) != hipSuccess) st = QASR_ERR_HIP;
  if (st == QASR_OK) st = forward_impl(e, x, y, workspace, workspace_bytes, (hipStream_t)stream, how);
  if (st == QASR_OK && hipEventSynchronize(ev[n]) != hipSuccess) st = QASR_ERR_HIP;
  float per_event_ms = 0.f;
  if (st == QASR_OK) {
    float plain = 0.f, evented = 0.f;
    if (hipEventElapsedTime(&plain, cal[0], cal[1]) != hipSuccess || hipEventElapsedTime(&evented, ev[0], ev[n]) != hipSuccess)
      st = QASR_ERR_HIP;
    const size_t launches = (size_t)std::count(began.begin(), began.end(), 1);
    per_event_ms = evented > plain ? (evented - plain) / (float)launches : 0.f;
  }
  began[n] = 1;
  for (size_t i = 0; i < n && st == QASR_OK; ++i) {
    op_ms[i] = 0.f;
    if (!began[i]) continue;                      // (part of the launch before)
    size_t next = i + 1;
    while (!began[next]) ++next;
    if (hipEventElapsedTime(&op_ms[i], ev[i], ev[next]) != hipSuccess) st = QASR_ERR_HIP;
    op_ms[i] = op_ms[i] > per_event_ms ? op_ms[i] - per_event_ms : 0.f;
  }
  for (hipEvent_t v : cal)
    if (v) (void)hipEventDestroy(v);
  for (hipEvent_t v : ev)
    if (v) (void)hipEventDestroy(v);
  return st;
}

struct qasr_encoder_graph {
  hipGraphExec_t exec = nullptr;
  // Launching a graph costs the host 16 us however small it is, a kernel by itself 3 us: forwards of up to
  // kDirectKernels kernels are enqueued one by one (exec stays null), which also runs them sooner.
  const qasr_encoder* e = nullptr;
  const int8_t* x = nullptr;
  int8_t* y = nullptr;
  void* workspace = nullptr;
  size_t workspace_bytes = 0;
};
static constexpr size_t kDirectKernels = 4;

qasr_status qasr_encoder_graph_create(const qasr_encoder* e, const int8_t* x, int8_t* y, void* workspace,
                                      size_t workspace_bytes, qasr_encoder_graph** out) {
  if (!e || !out) return QASR_ERR_NULL;
  *out = nullptr;
  hipStream_t cap = nullptr;
  if (hipStreamCreate(&cap) != hipSuccess) return QASR_ERR_HIP;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  // One ordinary forward first: argument checks, and the one-time per-kernel set-up (attribute
  // calls) that must not happen while the stream is capturing.
  qasr_status st = forward_impl(e, x, y, workspace, workspace_bytes, cap);
  if (st == QASR_OK && hipStreamSynchronize(cap) != hipSuccess) st = QASR_ERR_HIP;
  if (st == QASR_OK) {
    if (hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal) != hipSuccess) {
      st = QASR_ERR_HIP;
    } else {
      st = forward_impl(e, x, y, workspace, workspace_bytes, cap);
      const hipError_t ee = hipStreamEndCapture(cap, &graph);      // always ends the capture
      if (st == QASR_OK && (ee != hipSuccess || !graph)) st = QASR_ERR_HIP;
    }
  }
  size_t nodes = 0;
  if (st == QASR_OK && hipGraphGetNodes(graph, nullptr, &nodes) != hipSuccess) st = QASR_ERR_HIP;
  const bool direct = nodes <= kDirectKernels;
  if (st == QASR_OK && !direct && hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0) != hipSuccess) st = QASR_ERR_HIP;
  if (graph) (void)hipGraphDestroy(graph);
  (void)hipStreamDestroy(cap);
  if (st != QASR_OK) return st;
  qasr_encoder_graph* g = new (std::nothrow) qasr_encoder_graph();
  if (!g) {
    if (exec) (void)hipGraphExecDestroy(exec);
    return QASR_ERR_HIP;
  }
  g->exec = exec;
  g->e = e; g->x = x; g->y = y; g->workspace = workspace; g->workspace_bytes = workspace_bytes;
  *out = g;
  return QASR_OK;
}

qasr_status qasr_encoder_graph_launch(qasr_encoder_graph* g, void* stream) {
  if (!g) return QASR_ERR_NULL;
  if (!g->exec) return forward_impl(g->e, g->x, g->y, g->workspace, g->workspace_bytes, (hipStream_t)stream);
  const hipError_t e = hipGraphLaunch(g->exec, (hipStream_t)stream);
  return e == hipSuccess ? QASR_OK : hip_status(e);
}

void qasr_encoder_graph_destroy(qasr_encoder_graph* g) {
  if (!g) return;
  if (g->exec) (void)hipGraphExecDestroy(g->exec);
  delete g;
}

void qasr_encoder_destroy(qasr_encoder* e) {
  if (!e) return;
  if (e->packed) (void)hipFree(e->packed);
  if (e->sep_images) (void)hipFree(e->sep_images);
  if (e->toeplitz) (void)hipFree(e->toeplitz);
  for (qasr_encoder::TeamRun& r : e->runs) {
    if (r.ops_dev) (void)hipFree(r.ops_dev);
    if (r.ctl) (void)hipFree(r.ctl);
  }
  qasr_encoder_destroy(e->dense);
  delete e;
}

void qasr_tuning_reload(void) { qasr::tuning_reload(); }

const char* qasr_last_hip_error(void) { return hipGetErrorName(g_last_hip); }

const char* qasr_status_string(qasr_status st) {
  switch (st) {
    case QASR_OK: return "ok";
    case QASR_ERR_NULL: return "required pointer is NULL";
    case QASR_ERR_SHAPE: return "invalid shape";
    case QASR_ERR_PARAM: return "invalid parameter";
    case QASR_ERR_UNSUPPORTED: return "unsupported grouping";
    case QASR_ERR_ALIAS: return "output overlaps an input";
    case QASR_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case QASR_ERR_HIP: return "HIP runtime error";
  }
  return "unknown status";
}

}  // extern "C"
