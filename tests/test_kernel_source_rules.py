"""Source-level rules of the kernels that count their own vector-memory requests (csrc/vmem.hpp).

The compiler knows nothing of a load issued through the inline-assembly wrappers: nothing stops a
wave from ending, or a function from returning into code that reuses the registers or the LDS
rows, while such a load is still in flight.  The rules checked here, on the text of the sources:

  1. every function that issues such loads reaches `wait_vm<0>()` after its last request, and no
     `return` between the first request and the end comes without one; functions that only ask, for the caller's registers,
     are named (ASKS), and a call of one counts as a request of its caller;
  2. those sources never read a layer operand through a plain dereference (`p.m[c]`, `*p.bias`):
     a load the compiler does see makes it wait for everything outstanding, and a hand count that
     was right becomes a stall (or, with its registers reassigned, wrong data).
"""
import os
import re

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2103_16827_amd", "csrc")

# functions that leave what they ask for on its way (a kernel's ring, its constants): pw_chain.hip, sep_body.hpp
ASKS = ("load_step", "load_steps", "items", "load_by_hand")
LOADS = (r"\b(?:direct_load16_scope\s*<[^>]*>|direct_load16_dev|direct_load16|direct_load4|gload16|gload8|gload4|gload_i8|bload16"
         r"|gload16_into\s*<[^;]*?>|gload4_into|(?:load_step|load_steps|items)\s*<[^;()]*>|load_by_hand)\s*\(")
WAIT0 = r"\bwait_vm\s*<\s*0\s*>\s*\(\s*\)"
OPERANDS = r"(?:bias|m|s|w|x|res|act_lut)"


def strip_comments(text):
    text = re.sub(r"/\*.*?\*/", lambda m: " " * len(m.group(0)), text, flags=re.S)
    return re.sub(r"//[^\n]*", lambda m: " " * len(m.group(0)), text)


def sources():
    out = {}
    for name in sorted(os.listdir(CSRC)):
        if name.endswith((".hip", ".hpp")) and name != "vmem.hpp":
            out[name] = strip_comments(open(os.path.join(CSRC, name)).read())
    return out


def functions(text):
    """(name, body) of every __global__ / __device__ function definition in `text`."""
    found = []
    for m in re.finditer(r"__(?:global|device)__", text):
        i = text.find("(", m.end())
        # the parameter list: the first parenthesis that is not part of an attribute or launch bound
        while i >= 0:
            head = text[m.end():i]
            if re.search(r"(?:__launch_bounds__|__attribute__\s*\(?)\s*$", head):
                depth, j = 0, i
                while True:
                    depth += text[j] == "("
                    depth -= text[j] == ")"
                    j += 1
                    if depth == 0:
                        break
                i = text.find("(", j)
                continue
            break
        if i < 0:
            continue
        name = re.findall(r"(\w+)\s*$", text[m.end():i])
        depth, j = 0, i
        while True:
            depth += text[j] == "("
            depth -= text[j] == ")"
            j += 1
            if depth == 0:
                break
        k = j
        while k < len(text) and text[k] in " \n\t":
            k += 1
        if k >= len(text) or text[k] != "{":
            continue                      # a declaration
        depth, e = 0, k
        while True:
            depth += text[e] == "{"
            depth -= text[e] == "}"
            e += 1
            if depth == 0:
                break
        found.append((name[0] if name else "?", text[k:e]))
    return found


def lambda_spans(body):
    """Character ranges of the lambda bodies inside a function body (a `return` there leaves the
    lambda, not the function)."""
    spans = []
    for m in re.finditer(r"\[[&=]?\]\s*\(", body):
        depth, j = 0, m.end() - 1
        while True:
            depth += body[j] == "("
            depth -= body[j] == ")"
            j += 1
            if depth == 0:
                break
        k = body.find("{", j)
        if k < 0 or ";" in body[j:k]:
            continue
        depth, e = 0, k
        while True:
            depth += body[e] == "{"
            depth -= body[e] == "}"
            e += 1
            if depth == 0:
                break
        spans.append((k, e))
    return spans


def function_returns(body):
    spans = lambda_spans(body)
    return [r.start() for r in re.finditer(r"\breturn\b", body) if not any(a <= r.start() < b for a, b in spans)]


def test_the_splitter_sees_the_kernels():
    src = sources()
    names = {n for t in src.values() for n, _ in functions(t)}
    for want in ("pw_pipe_kernel", "pw_pipe_tile", "dw_pipe_kernel", "pw_tile_kernel", "team_kernel", "conv_pipe_kernel", "conv_few_kernel", "pw_chain_kernel", *ASKS):
        assert want in names, (want, sorted(names))


def undrained(name, body):
    """What is wrong with a function that issues hand-counted loads, or None (False: it issues none)."""
    loads = [m.start() for m in re.finditer(LOADS, body)]
    if not loads:
        return False
    waits = [m.start() for m in re.finditer(WAIT0, body)]
    if name in ASKS:
        return "a return where only requests are made" if function_returns(body) else None
    if not (waits and waits[-1] > loads[-1]):
        return "no wait_vm<0>() after its last request"
    for r in function_returns(body):
        before = [q for q in loads if q < r]
        if before and not any(before[-1] < w < r for w in waits):    # (else it leaves before anything was requested)
            return "a return after a request without wait_vm<0>() in between"
    return None


def test_every_function_with_hand_counted_loads_drains_them_before_it_ends():
    checked = []
    for fname, text in sources().items():
        for name, body in functions(text):
            wrong = undrained(name, body)
            assert not wrong, f"{fname}:{name}: {wrong}"
            if wrong is None:
                checked.append(f"{fname}:{name}")
    # the kernels known to use the wrappers are all among the checked ones
    for want in ("pw_pipe_tile", "dw_pipe_kernel", "pw_tile_kernel", "conv_pipe_kernel", "conv_few_kernel", "pw_chain_kernel", *ASKS):
        assert any(c.endswith(":" + want) for c in checked), checked


def test_requests_into_the_callers_registers_are_seen():
    """Every wrapper of vmem.hpp counts as a request, and a function that only asks and is not known to is refused."""
    vmem = strip_comments(open(os.path.join(CSRC, "vmem.hpp")).read())
    asks = [n for n, body in functions(vmem) if re.search(r"(?:global|buffer)_load", body) or n.startswith("direct_load")]
    assert {"gload16_into", "gload4_into", "gload16", "direct_load4"} <= set(asks)
    for n in asks:
        call = f"{n}<{'true' if 'scope' in n else 'I * 8'}>(r, p);" if n in ("gload16_into", "direct_load16_scope") else f"{n}(r, p);"
        assert re.search(LOADS, call), n
    (name, body), = functions("template <int I> __device__ void other(v4i& r) { gload16_into<(I & 3) * 1024>(r, p, o); }")
    assert undrained(name, body) and undrained("load_step", body) is None
    assert undrained("load_step", "{ if (a) return; gload4_into(r, p); }")
    # ... and what asks through one that is known to
    assert undrained("k", "{ load_steps<0, D / 2>(wb, w0, w1, wlane); }") and undrained("k", "{ items<MT, true, 0>(acc, wb, ar, a0, n, w0, w1, l); }")
    (kernel,) = [b for n, b in functions(sources()["pw_chain.hip"]) if n == "pw_chain_kernel"]
    assert undrained("pw_chain_kernel", kernel) is None
    assert undrained("pw_chain_kernel", kernel.replace("wait_vm<0>();", ""))


def test_the_checker_catches_a_missing_drain():
    bad = """
    __global__ void k(const int* p) {
      v4i a = gload16(p);
      wait_vm<0>();
      v4i b = gload16(p + 4);
      if (threadIdx.x == 0) return;
    }
    """
    (name, body), = functions(bad)
    loads = [m.start() for m in re.finditer(LOADS, body)]
    waits = [m.start() for m in re.finditer(WAIT0, body)]
    assert name == "k" and len(loads) == 2 and len(waits) == 1
    assert not waits[-1] > loads[-1]
    assert len(function_returns(body)) == 1
    with_lambda = "__device__ void f() { auto g = [&](int i) __attribute__((always_inline)) { return i; }; gload4(0); wait_vm<0>(); }"
    (_, body2), = functions(with_lambda)
    assert function_returns(body2) == []


def test_no_plain_dereference_of_layer_operands_where_loads_are_hand_counted():
    for fname, text in sources().items():
        if not re.search(LOADS, text):
            continue
        # (the layer's parameter block is called p in every kernel, v in the team kernel's layer view)
        for pat in (rf"\b[pv](?:\.|->){OPERANDS}\s*\[", rf"\*\s*\(?\s*[pv](?:\.|->){OPERANDS}\b(?!\s*[?!=])"):
            for m in re.finditer(pat, text):
                line = text.count("\n", 0, m.start()) + 1
                raise AssertionError(f"{fname}:{line}: operand read outside the vmem.hpp wrappers: "
                                     f"{text[m.start():m.end() + 20]!r}")
    assert re.search(rf"\b[pv](?:\.|->){OPERANDS}\s*\[", "x = p.m[co];") and re.search(
        rf"\*\s*\(?\s*[pv](?:\.|->){OPERANDS}\b(?!\s*[?!=])", "int b = *p.bias;")


def handover_orders(body):
    """Positions of a split contraction's steps: partial sums stored, all waves' stores complete, arrival counted
    with release order, acquire fence of the last workgroup, barrier, the others' sums loaded."""
    steps = [r"raw_buffer_store_b128\s*\([^;]*\bmine\b", r"s_waitcnt vmcnt\(0\)", r"__syncthreads\s*\(\s*\)",
             r"__hip_atomic_fetch_add\s*\([^;]*__ATOMIC_(?:RELEASE|ACQ_REL)\s*,\s*__HIP_MEMORY_SCOPE_AGENT",
             r"__builtin_amdgcn_fence\s*\(\s*__ATOMIC_ACQUIRE\s*,\s*\"agent\"\s*\)", r"__syncthreads\s*\(\s*\)",
             r"raw_buffer_load_b128\s*\([^;]*\bfrom\b"]
    at, found = 0, []
    for s in steps:
        m = re.compile(s).search(body, at)
        if not m:
            return None
        at = m.end()
        found.append(m.start())
    return found


def test_partial_sums_are_handed_over_with_release_and_acquire():
    """Workgroups of one tile may run on different dies, whose caches see each other's writes only through
    device-scope release and acquire."""
    (body,) = [b for n, b in functions(sources()["conv_pipe.hip"]) if n == "conv_pipe_kernel"]
    assert handover_orders(body)
    assert not handover_orders(body.replace("__ATOMIC_RELEASE", "__ATOMIC_RELAXED"))
    assert not handover_orders(body.replace("__ATOMIC_ACQUIRE", "__ATOMIC_RELAXED"))
    for name, text in sources().items():          # no other kernel counts arrivals with less
        if name in ("team.hip",):                 # (bounded polls of one die's team, off by default)
            continue
        assert not re.search(r"__hip_atomic_fetch_add\s*\([^;]*__ATOMIC_RELAXED", text), name
