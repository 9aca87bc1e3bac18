"""CPU replay of the hand-kept bookkeeping of chains of pointwise layers (csrc/pw_chain.hip): one stream of weights over layers,
passes and blocks, requests into LDS that overlays what later layers write, one barrier per layer.  tests/sim/chain_sim_main.cpp
lists what is checked; test_pw_pipe_host_sim.py says how such a replay works."""
import os
import re
import subprocess

import pytest

from test_pw_pipe_host_sim import CLANG, CSRC, SIM, generate

pytestmark = pytest.mark.skipif(not os.path.exists(CLANG), reason="no host clang beside the HIP toolchain")


def span(text, begin, end):
    m = re.search(begin + r".*?" + end, text, flags=re.S)
    assert m, begin
    return m.group(0) + "\n"


def accesses(body, edits):
    """The kernel's own LDS accesses go through the recording stand-ins."""
    for pattern, stand_in, times in edits:
        body, n = re.subn(pattern, stand_in, body)
        assert n == times, (pattern, n)
    return body


def generate_chain(tmp, mutate=None):
    read = lambda name: open(os.path.join(CSRC, name)).read()
    strip = lambda t: re.sub(r"#(include|pragma once)[^\n]*\n", "", t)
    body, header = read("pw_chain.hip"), read("pw_chain.hpp")
    if mutate:
        body = mutate(body)
    body = accesses(strip(body), [
        (r"extern __shared__ [^;]*;", "unsigned char* const lds = sim::S().lds;", 1),
        (r'asm volatile\(""\s*::"s"[^;]*;', ";", 3),
        (r'asm volatile\("s_waitcnt lgkmcnt\(0\)" ::: "memory"\);', "", 1),
        (r"\*reinterpret_cast<v4i\*>\((lds \+ p\.buf[^=]*?|to \+ 16 \* lane)\) =\s*([^;]*);", r"sim_lds_write16(\1, \2);", 2),
        (r"v4i\* const c = reinterpret_cast<v4i\*>\(([^;]*)\);", r"unsigned char* const c = \1;", 1),
        (r"\*c = \(v4i\)\{0, 0, 0, 0\};", "sim_lds_write16(c, (v4i){0, 0, 0, 0});", 1),
        (r"\*c = keep_bytes\(\*c, ([^;]*)\);", r"sim_lds_write16(c, (v4i){0, 0, 0, 0});", 1),
        (r"\*reinterpret_cast<uint32_t\*>\((to \+ q \* 8192 \+ bk \* 256|o \+ 256 \* c[01])\) = ", r"SimWord{\1} = ", 4),
        (r"\*reinterpret_cast<const int32_t\*>\((cst[^;]*?)\)(?=[,;])", r"sim_lds_const(\1)", 6),
        (r"\*reinterpret_cast<const v4i\*>\((out \+ [^;]*) : 0\)\);", r"sim_lds_read16(\1 : 256 * c0));", 1),   # (what lanes without a row read is dropped)
        (r"\(int32_t\)table\[([^\]]*)\]", r"sim_table_code(table + (\1))", 1),
    ])
    assert "asm" not in re.sub(r'asm volatile\("" ::: "memory"\);', "", re.sub(r"//[^\n]*", "", body))
    left = [l for l in re.findall(r"\*reinterpret_cast<[^>]*>\([^\n]*", body) if "p.dw.img" not in l]
    assert left == [], left
    open(os.path.join(tmp, "pw_chain_stripped.hpp"), "w").write(
        "namespace qasr { struct SimWord { unsigned char* p; void operator=(uint32_t v) const { sim_lds_write4(p, v); } }; }\n" + body)

    sep, plan = read("sep_body.hpp"), read("sep.hip")
    small = accesses(span(sep, r"template <int CPW, int MT, int NA, bool RAGGED>\nstruct DwSmall \{", r"\n\};"), [
        (r"\*reinterpret_cast<const uint32_t\*>\((win [^;]*)\);", r"sim_lds_word(\1);", 1),
        (r"= \*reinterpret_cast<const v4i\*>\((wrow [^;]*)\);", r"= sim_lds_read16(\1);", 1),
        (r"(?s)  // \(the bias first.*?(?=  // NB blocks of 16 channels)", "", 1),       # (what the chain does itself)
    ])
    open(os.path.join(tmp, "sep_extract.hpp"), "w").write(
        "namespace qasr {\n" + span(read("sep.hpp"), r"struct DwParams \{", r"\n\};") + "namespace sep {\ntypedef unsigned v4u __attribute__((ext_vector_type(4)));\n"
        + "".join(span(sep, b, e) for b, e in ((r"constexpr int kStoreThrough", r";"), (r"constexpr int kWaves", r";"), (r"constexpr int kMaxUnits", r";"),
                                               (r"constexpr int row_loads\(", r"\n\}"), (r"inline int small_row_bytes\(", r"\n\}"),
                                               (r"uint32_t toeplitz_bytes\(", r"\}"),
                                               (r"template <int N>\nstruct Consts \{", r"\n\};")))
        + small + "}\n" + span(plan, r"struct Geometry \{", r"\nbool geometry\(.*?\n\}") + span(plan, r"bool x_ragged\(", r"\n") + span(plan, r"int units_of\(", r"\n\}")
        + span(plan, r"static void fill_dw\(", r"\n\}") + span(plan, r"bool dw_small_params\(", r"\n\}") + span(header, r"constexpr int kMaxChain", r";")
        + span(header, r"struct ChainLayer \{", r"\n\};") + span(header, r"struct ChainParams \{", r"\n\};") + span(header, r"struct ChainOp \{", r"\n\};") + "}\n")
    open(os.path.join(tmp, "divide_extract.hpp"), "w").write(
        "namespace qasr {\n" + span(read("common.hpp"), r"__device__ __forceinline__ int divide_uniform24", r"\n\}") + "}\n")
    generate(tmp)          # (ConvParams)


def build_and_run_chain(tmp, small=False):
    exe = os.path.join(tmp, "chain_sim")
    cmd = [CLANG, "-std=c++17", "-O0", "-g0", "-ftrivial-auto-var-init=zero", "-Wno-unknown-attributes", "-Wno-ignored-attributes", "-I", tmp, "-I", SIM, "-I", CSRC,
           os.path.join(SIM, "chain_sim_main.cpp"), "-o", exe]
    cmd += ["-DSIM_SMALL"] if small else ["-fsanitize=address,undefined", "-fno-sanitize=shift,signed-integer-overflow", "-fno-sanitize-recover=all"]
    c = subprocess.run(cmd, capture_output=True, text=True, timeout=900)
    assert c.returncode == 0, c.stderr[-6000:]
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:verify_asan_link_order=0", UBSAN_OPTIONS="halt_on_error=1")
    return subprocess.run([exe], capture_output=True, text=True, timeout=900, env=env)


def test_request_bookkeeping_of_chains_replays_cleanly(tmp_path):
    generate_chain(str(tmp_path))
    r = build_and_run_chain(str(tmp_path))
    assert r.returncode == 0, (r.stdout[-3000:], r.stderr[-3000:])
    assert "all cases passed" in r.stdout and r.stdout.count("ok ") >= 10, r.stdout


MISTAKES = {
    # a wait that allows one step too many, in the stream and at its end
    "stream": ("wait_vm<MORE ? 2 * (D - 1) : 2 * (D - 1 - st)>();", "wait_vm<MORE ? 2 * D : 2 * (D - 1 - st)>();"),
    "stream_end": ("wait_vm<MORE ? 2 * (D - 1) : 2 * (D - 1 - st)>();", "wait_vm<MORE ? 2 * (D - 1) : 2 * (D - st)>();"),
    # ... for the depthwise layer's rows and constants, for the tile and the layers' constants
    "rows": ("    wait_vm<D>();                                   // (and as many", "    wait_vm<D + 1>();  // (and as many"),
    "tile": ("  wait_vm<D>();                                     // tile, constants", "  wait_vm<D + 1>();  // tile, constants"),
    # no barrier between layers, or before the first
    "layers": ("    if (layer_end) barrier();\n", ""),
    "first": ("  barrier();\n  begin_pass();\n", "  begin_pass();\n"),
    # the depthwise layer's rows over the first layer's input, the constants over its taps
    "scratch": ("c.rows_off = 512 * 16 * MT;", "c.rows_off = 0;"),
    "constants": ("if (end > c.const_off) c.const_off = end;", ""),
    # one buffer instead of two; tiles that do not follow each other
    "buffers": ("unsigned char* const out = lds + p.buf[(cur.l + 1) & 1];", "unsigned char* const out = lds + p.buf[cur.l & 1];"),
    "tiles": ("ti * p.g_base + min(ti, p.g_more)", "ti * p.g_base"),
    # the stream asks on after its last block
    "drain": ("  items<MT, false, 0>(acc, wb, ar, a0, p.layer[cur.l].cin * 16, w0, w1, wlane);\n", "  items<MT, true, 0>(acc, wb, ar, a0, p.layer[cur.l].cin * 16, w0, w1, wlane);\n"),
}


@pytest.mark.parametrize("what", sorted(MISTAKES))
def test_the_replay_of_chains_catches_planted_mistakes(tmp_path, what):
    a, b = MISTAKES[what]

    def mutate(body):
        assert body.count(a) == 1, what
        return body.replace(a, b)
    generate_chain(str(tmp_path), mutate)
    r = build_and_run_chain(str(tmp_path), small=True)
    assert r.returncode != 0 and "SIM FAILURE" in r.stderr, (r.stdout[-2000:], r.stderr[-2000:])
