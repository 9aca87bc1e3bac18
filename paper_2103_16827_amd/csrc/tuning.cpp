// Environment overrides of the kernel choices (see tuning.hpp), parsed once.
#include "tuning.hpp"

#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <mutex>

namespace qasr {

namespace {

std::mutex g_mu;
Tuning g_tuning;
std::atomic<bool> g_loaded{false};

Tuning read_env() {
  Tuning t;
  t.no_pw_pipe = getenv("QASR_NO_PW_PIPE") != nullptr;
  t.no_conv_pipe = getenv("QASR_NO_CONV_PIPE") != nullptr;
  t.team = getenv("QASR_TEAM") != nullptr;
  t.cp_plain_order = getenv("QASR_CP_PLAIN_ORDER") != nullptr;
  t.no_pw_lean = getenv("QASR_NO_PW_LEAN") != nullptr;
  t.pw_lean_force = getenv("QASR_PW_LEAN") != nullptr;
  t.pw_lean_no_res = getenv("QASR_PW_LEAN_NO_RES") != nullptr;
  t.pwp_nopipe = getenv("QASR_PWP_NOPIPE") != nullptr;
  if (const char* e = getenv("QASR_PWP_MT")) t.pwp_mt = atoi(e);
  if (const char* e = getenv("QASR_PWP_SPLIT")) t.pwp_split = atoi(e);
  if (const char* e = getenv("QASR_DWP")) {
    int r = 0, s = 0;
    if (sscanf(e, "%d,%d", &r, &s) == 2) { t.dwp_r = r; t.dwp_s = s; }
  }
  if (const char* e = getenv("QASR_DW_R")) t.dw_r = atoi(e);
  if (const char* e = getenv("QASR_CP_TILE")) {
    int mt = 0, nt = 0, kg = 0, s = 0;
    if (sscanf(e, "%d,%d,%d,%d", &mt, &nt, &kg, &s) >= 1) { t.cp_mt = mt; t.cp_nt = nt; t.cp_kg = kg; t.cp_s = s; }
  }
  t.no_conv_few = getenv("QASR_NO_CONV_FEW") != nullptr;
  t.conv_few_force = getenv("QASR_CONV_FEW") != nullptr;
  if (const char* e = getenv("QASR_CF")) {
    int mt = 0, wc = 0, nt = 0;
    if (sscanf(e, "%d,%d,%d", &mt, &wc, &nt) >= 1) { t.cf_mt = mt; t.cf_wc = wc; t.cf_nt = nt || !wc ? nt : 2; }
  }
  t.no_pw_multi = getenv("QASR_NO_PW_MULTI") != nullptr;
  t.pw_multi_force = getenv("QASR_PW_MULTI") != nullptr;
  t.no_pw_chain = getenv("QASR_NO_PW_CHAIN") != nullptr;
  t.pw_chain_force = getenv("QASR_PW_CHAIN") != nullptr;
  if (const char* e = getenv("QASR_CHAIN_MT")) t.chain_mt = atoi(e);
  t.no_sep = getenv("QASR_NO_SEP") != nullptr;
  t.no_pw_wide = getenv("QASR_NO_PW_WIDE") != nullptr;
  t.pw_wide_force = getenv("QASR_PW_WIDE") != nullptr;
  if (const char* e = getenv("QASR_PWW")) {
    int mt = 0, ks = 0;
    if (sscanf(e, "%d,%d", &mt, &ks) >= 1) { t.pww_mt = mt; t.pww_ks = ks; }
  }
  if (const char* e = getenv("QASR_SEP")) {
    int mt = 0, nt = 0, ks = 0;
    if (sscanf(e, "%d,%d,%d", &mt, &nt, &ks) >= 1) { t.sep_mt = mt; t.sep_nt = nt; t.sep_ks = ks; }
  }
  if (const char* e = getenv("QASR_PWT_MT")) t.pwt_mt = atoi(e);
  if (const char* e = getenv("QASR_SLOT_DEPTH")) {
    const int d = atoi(e);
    if (d >= 0 && d <= 16) t.slot_depth = d;
  }
  return t;
}

}  // namespace

const Tuning& tuning() {
  if (!g_loaded.load(std::memory_order_acquire)) {
    std::lock_guard<std::mutex> lk(g_mu);
    if (!g_loaded.load(std::memory_order_relaxed)) {
      g_tuning = read_env();
      g_loaded.store(true, std::memory_order_release);
    }
  }
  return g_tuning;
}

void tuning_reload() {
  std::lock_guard<std::mutex> lk(g_mu);
  g_tuning = read_env();
  g_loaded.store(true, std::memory_order_release);
}

}  // namespace qasr
