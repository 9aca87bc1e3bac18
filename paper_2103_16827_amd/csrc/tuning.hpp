// Tuning overrides of the kernel choices, read from the environment ONCE (at first use) instead of
// on every launch; tuning_reload() reads them again (tests and sweeps that change the environment
// of a running process call it through qasr_tuning_reload).  0 / false = no override.
//   QASR_NO_PW_PIPE, QASR_NO_CONV_PIPE      fall through to the next kernel family
//   QASR_PWP_MT, QASR_PWP_SPLIT             pw_pipe: groups per tile, workgroups per tile
//   QASR_DWP = "R,S"                        dw_pipe: rows per iteration, batch splits
//   QASR_DW_R                               dw_mfma: strips per wave
//   QASR_CP_TILE = "MT,NT[,KG[,S]]"         conv_pipe: tile, wave groups the taps and workgroups the chunks are split over
//   QASR_NO_CONV_FEW, QASR_CONV_FEW         conv_few: never / wherever it can
//   QASR_CF = "MT,WC,NT"                    conv_few: groups per tile, column waves, 16-channel columns of each (0: free)
//   QASR_CP_PLAIN_ORDER                     conv_pipe: tile = workgroup index (no per-XCD runs of the channel-major order)
//   QASR_PWT_MT                             pw_tile: groups per tile
//   QASR_PWP_NOPIPE                         pw_pipe: no epilogue under the next pass's products
//   QASR_PW_LEAN                            pw_pipe: the lean form for every layer it can take, whatever the launch size
//   QASR_PW_LEAN_NO_RES                     pw_pipe: layers with a residual operand keep the pipelined form
//   QASR_NO_PW_LEAN                         pw_pipe: never the lean form (one pass per workgroup, two workgroups per unit)
//   QASR_SLOT_DEPTH                         encoder: an op's output avoids the buffers the last N ops touched
//                                           (default 4; 0 = the caller's slots are the buffers)
//   QASR_NO_PW_WIDE, QASR_PW_WIDE            pw_wide: never / wherever it can
//   QASR_NO_PW_MULTI, QASR_PW_MULTI         encoder: several pointwise layers in one launch: never / wherever possible
//   QASR_NO_PW_CHAIN, QASR_PW_CHAIN         encoder: chains of pointwise layers in one launch: never / wherever possible
//   QASR_CHAIN_MT                           the same: groups per tile
//   QASR_PWW = "MT,KS"                      pw_wide: groups per tile, wave groups over the input channels (0: free)
//   QASR_NO_SEP                             encoder: no depthwise + pointwise pair in one launch
//   QASR_SEP = "MT,NT[,KS]"                 the same: groups per tile, 16-channel columns per wave (0: free), wave groups over
//                                           the input channels (1 where NT is given alone)
//   QASR_TEAM                               encoder: plan runs of layers for the persistent team kernel
//                                           (experimental, off unless set)
#pragma once

namespace qasr {

struct Tuning {
  bool no_pw_pipe = false, no_conv_pipe = false, team = false, cp_plain_order = false, no_pw_lean = false, pw_lean_force = false, pw_lean_no_res = false, pwp_nopipe = false, no_sep = false, no_pw_wide = false, pw_wide_force = false, no_conv_few = false, conv_few_force = false, no_pw_multi = false, pw_multi_force = false, no_pw_chain = false, pw_chain_force = false;
  int pwp_mt = 0, pwp_split = 0;
  int dwp_r = 0, dwp_s = 0;
  int dw_r = 0;
  int cp_mt = 0, cp_nt = 0, cp_kg = 0, cp_s = 0, cf_mt = 0, cf_wc = 0;
  int pwt_mt = 0;
  int sep_mt = 0, sep_nt = 0, sep_ks = 0, pww_mt = 0, pww_ks = 0, chain_mt = 0;
  int slot_depth = 4;
  int cf_nt = 0;
};

const Tuning& tuning();
void tuning_reload();

}  // namespace qasr
