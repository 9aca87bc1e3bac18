"""Performance cases of the integer-only ASR encoder library.

Each case is one thing a program that uses the library does through its public entry points, with
the sizes of the benchmark networks (qasr_workloads) and of ordinary speech data around them.  Speech
is 100 feature frames per second, so an utterance of 1 to 30 seconds is 100 to 3000 frames; front
ends either leave the frame count as it falls or round it up to a multiple of 16.  Weights, scales and
inputs follow the distributions of qasr_workloads.draw_net_params / draw_input, drawn on the GPU.

  kind "net"        a whole encoder: qasr_encoder_forward, _graph_launch or _forward_f32
  kind "layer"      one layer by itself: qasr_conv1d_int8 with packed weights
  kind "softmax"    attention probabilities from integer logits: qasr_softmax_int32
  kind "calibrate"  offline calibration of one layer: qasr_observe_minmax and qasr_fold_bn_quantize
"""
import math

import torch

import paper_2103_16827_amd as Q
import qasr_workloads as W
from paper_2103_16827_amd.binding import make_desc


def listed():
    return [
        # One separable module on two seconds of one utterance: the smallest call, all latency.
        {"name": "module_b1", "kind": "net", "net": "module", "B": 1, "T": 200, "entry": "forward"},
        # Live transcription of one 16 s utterance with the small network, replayed as a graph.
        {"name": "quartznet5x5_b1", "kind": "net", "net": "quartznet5", "B": 1, "T": 1600, "entry": "graph"},
        # Batch transcription with the full network: the benchmark's headline workload.
        {"name": "quartznet15x5_b32", "kind": "net", "net": "quartznet15", "B": 32, "T": 1600, "entry": "graph"},
        # One utterance as it falls (12.37 s), float features in and float logits out.
        {"name": "quartznet15x5_b1_odd", "kind": "net", "net": "quartznet15", "B": 1, "T": 1237, "entry": "f32"},
        # A server's batch of 8, padded to a multiple of 16 frames (552 frames after the stride).
        {"name": "quartznet10x5_b8", "kind": "net", "net": "quartznet10", "B": 8, "T": 1104, "entry": "forward"},
        # Batch transcription with the dense network: the largest amount of arithmetic.
        {"name": "jasper_b16", "kind": "net", "net": "jasper", "B": 16, "T": 1600, "entry": "graph"},
        # The dense-residual variant on two utterances of odd length.
        {"name": "jasper_dr_b2_odd", "kind": "net", "net": "jasper_dr", "B": 2, "T": 811, "entry": "forward"},
        # Conformer-shaped linear layers on 16 utterances of 16 s after the 4x subsampling.
        {"name": "conformer_b16", "kind": "net", "net": "conformer", "B": 16, "T": 400, "entry": "graph"},
        # The same with its integer Swish and GLU, on utterances of odd length.
        {"name": "conformer_act_b8_odd", "kind": "net", "net": "conformer_act", "B": 8, "T": 387, "entry": "forward"},
        # Attention probabilities of one layer: 16 utterances, 8 heads, 400 x 400 scores.
        {"name": "softmax_attention", "kind": "softmax", "rows": 51200, "L": 400},
        # One pointwise layer with a residual operand, for a program that chains layers by itself.
        {"name": "layer_pw_b8", "kind": "layer", "layer": "pw", "B": 8, "Cin": 512, "Cout": 512, "T": 800,
         "k": 1, "dilation": 1, "res": True, "relu": True},
        # Calibration of one dense layer: extremes of a batch of activations, folding of its weights.
        {"name": "calibrate_dense", "kind": "calibrate", "B": 16, "C": 640, "T": 800, "Cout": 768, "k": 25},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


# network -> (utterance lengths in frames, largest batch, largest batch x frames)
_NETS = {
    "module": ((50, 3000), 32, 51200),
    "quartznet5": ((100, 3000), 32, 51200),
    "quartznet10": ((100, 3000), 32, 51200),
    "quartznet15": ((100, 3000), 32, 51200),
    "jasper": ((100, 2000), 8, 4800),
    "jasper_dr": ((100, 2000), 8, 3200),
    "conformer": ((25, 750), 32, 6400),
    "conformer_act": ((25, 750), 32, 6400),
}


def _frames(rng, lo, hi):
    """An utterance length: as it falls, or rounded up to a multiple of 16 by the front end."""
    T = _log_int(rng, lo, hi)
    return (T + 15) // 16 * 16 if rng.random() < 0.5 else T


def draw(rng):
    kind = rng.choices(["net", "layer", "softmax", "calibrate"], [12, 5, 2, 1])[0]
    if kind == "net":
        net = rng.choice(sorted(_NETS))
        (lo, hi), most, total = _NETS[net]
        T = _frames(rng, lo, hi)
        B = _log_int(rng, 1, max(1, min(most, total // T)))
        return {"kind": "net", "net": net, "B": B, "T": T, "entry": rng.choice(["forward", "graph", "f32"])}
    if kind == "layer":
        layer = rng.choice(["dw", "pw", "dense"])
        T = _frames(rng, 50, 1500)
        B = _log_int(rng, 1, max(1, min(32, (25600 if layer != "dense" else 6400) // T)))
        if layer == "dw":
            C = rng.choice([256, 512, 1024])
            k, dil = rng.choice([(31, 1), (33, 1), (39, 1), (51, 1), (63, 1), (75, 1), (87, 2)])
            return {"kind": "layer", "layer": "dw", "B": B, "Cin": C, "Cout": C, "T": T, "k": k, "dilation": dil,
                    "res": False, "relu": False}
        widths = [256, 384, 512, 640, 768, 1024] + ([2048] if layer == "pw" else [])
        Cin, Cout = rng.choice(widths), rng.choice(widths)
        k = 1 if layer == "pw" else rng.choice([3, 11, 13, 17, 21, 25])
        return {"kind": "layer", "layer": layer, "B": B, "Cin": Cin, "Cout": Cout, "T": T, "k": k, "dilation": 1,
                "res": rng.random() < 0.3, "relu": rng.random() < 0.7}
    if kind == "softmax":
        L = _log_int(rng, 16, 4096)
        return {"kind": "softmax", "rows": _log_int(rng, 64, min(65536, (1 << 25) // L)), "L": L}
    T = _frames(rng, 50, 1500)
    return {"kind": "calibrate", "B": _log_int(rng, 1, 16), "C": rng.choice([256, 512, 768, 1024]), "T": T,
            "Cout": rng.choice([256, 512, 768, 1024]), "k": rng.choice([1, 11, 25])}


def _net_spec(case):
    name, B, T = case["net"], case["B"], case["T"]
    if name == "module":
        return W.separable_module(B, 256, T, 33)
    if name.startswith("quartznet"):
        return W.quartznet(B, T, {"5": 1, "10": 2, "15": 3}[name[len("quartznet"):]], 2)
    if name.startswith("jasper"):
        return W.jasper(B, T, 3, dense_residual=name == "jasper_dr")
    return W.conformer_shaped(B, T, 4, nonlinear=name == "conformer_act")


class _Draw:
    """Seeded draws on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)

    def ints(self, shape, lo, hi, dtype):
        return torch.randint(lo, hi + 1, shape, generator=self.g, dtype=dtype, device="cuda")

    def normal(self, shape, mean=0.0, std=1.0):
        return torch.randn(shape, generator=self.g, device="cuda") * std + mean

    def layer(self, Cout, per, k, bias=True):
        """(w, bias, m, s) with the distributions of qasr_workloads.draw_net_params."""
        return (self.ints((Cout, per, k), -127, 127, torch.int8),
                self.ints((Cout,), -(1 << 16), 1 << 16, torch.int32) if bias else None,
                self.ints((Cout,), 1 << 30, (1 << 31) - 2, torch.int32), self.ints((Cout,), 36, 44, torch.int32))


def prepare(case, seed):
    d = _Draw(seed)
    st = {"case": case}
    if case["kind"] == "net":
        net = _net_spec(case)
        ops = []
        for o in net.ops:
            w, bias, m, s = d.layer(o.Cout, 1 if o.depthwise else o.Cin, o.k, o.has_bias)
            # an activation's output rescale keeps about the scale of its input, 4 to 8 over 127 codes
            act = Q.make_act(o.act, Q.iexp_init(6.0 / 127.0, 8), 3 << 29, 45) if o.act else None
            desc = make_desc(net.B, o.Cin, o.Cout, o.Tin, o.k, o.stride, o.dilation, o.pad_left, o.pad_right, o.groups,
                             o.x_batch_stride, 0, o.flags)
            ops.append((desc, w, bias, m, s, o.in_slot, o.res_slot, o.out_slot, act, list(o.more_res)))
        enc = st["encoder"] = Q.Encoder(ops, net.n_slots)
        f32 = case["entry"] == "f32"
        shape = (net.B, net.Cin, net.Tin)
        x = d.normal(shape) if f32 else d.ints(shape, -128, 127, torch.int8)   # features are normalised per channel
        y = torch.empty((net.B, net.Cout, net.Tout), dtype=torch.float32 if f32 else torch.int8, device="cuda")
        need = enc.workspace_bytes_f32 if f32 else enc.workspace_bytes
        ws = torch.empty(max(need, 256), dtype=torch.int8, device="cuda")
        st.update(x=x, y=y, ws=ws)
        if case["entry"] == "graph":
            st["graph"] = enc.graph(x, y, ws)
    elif case["kind"] == "layer":
        B, Cin, Cout, T, k, dil = (case[n] for n in ("B", "Cin", "Cout", "T", "k", "dilation"))
        dw = case["layer"] == "dw"
        tot = dil * (k - 1)
        w, bias, m, s = d.layer(Cout, 1 if dw else Cin, k, not dw)
        st.update(x=d.ints((B, Cin, T), -128, 127, torch.int8), bias=bias, m=m, s=s,
                  y=torch.empty((B, Cout, T), dtype=torch.int8, device="cuda"),
                  res=d.ints((B, Cout, T), -128, 127, torch.int8) if case["res"] else None)
        desc = make_desc(B, Cin, Cout, T, k, 1, dil, tot // 2, tot - tot // 2, Cin if dw else 1, 0, 0,
                         Q.FLAG_RELU if case["relu"] else 0)
        packed = torch.empty(Q.packed_weight_bytes(desc), dtype=torch.int8, device="cuda")
        st["w"] = Q.pack_weights(desc, w, packed)
        desc.flags |= Q.FLAG_W_PACKED
        st["desc"] = desc
        torch.cuda.current_stream().synchronize()      # the plain weights go away here
    elif case["kind"] == "softmax":
        x = d.normal((case["rows"], case["L"]), std=250.0).round().to(torch.int32)   # scores at scale 0.01
        st.update(x=x, e=Q.iexp_init(0.01, 2), y=torch.empty(x.shape, dtype=torch.int8, device="cuda"))
    else:
        C, Cout, k = case["C"], case["Cout"], case["k"]
        st.update(x=d.normal((case["B"], C, case["T"])), w=d.normal((Cout, C, k), std=(C * k) ** -0.5),
                  gamma=d.normal((Cout,), 1.0, 0.1), beta=d.normal((Cout,), 0.0, 0.1), mean=d.normal((Cout,), 0.0, 0.1),
                  var=d.normal((Cout,), 1.0, 0.1).abs() + 0.01,
                  minmax=torch.tensor([float("inf"), float("-inf")], device="cuda"),
                  q_w=torch.empty((Cout, C, k), dtype=torch.int8, device="cuda"),
                  S_w=torch.empty(Cout, device="cuda"),
                  **{n: torch.empty(Cout, dtype=torch.int32, device="cuda") for n in ("bias", "m", "s")})
    return st


def run(st):
    case = st["case"]
    if case["kind"] == "net":
        if case["entry"] == "graph":
            return st["graph"].launch()
        if case["entry"] == "f32":
            return st["encoder"].forward_f32(st["x"], 4.0, 0.05, st["y"], st["ws"])
        return st["encoder"].forward(st["x"], st["y"], st["ws"])
    if case["kind"] == "layer":
        return Q.conv1d_int8(st["desc"], st["x"], st["w"], st["bias"], st["m"], st["s"], st["res"], st["y"])
    if case["kind"] == "softmax":
        return Q.softmax_int32(st["e"], st["x"], st["y"])
    Q.observe_minmax(st["x"], st["minmax"])
    Q.fold_bn_quantize(st["w"], None, st["gamma"], st["beta"], st["mean"], st["var"], 1e-5, 4.0 / 127, 6.0 / 127,
                       st["q_w"], st["bias"], st["m"], st["s"], st["S_w"])
    return {n: st[n] for n in ("minmax", "q_w", "bias", "m", "s", "S_w")}


def work(case):
    """Input, weights and per-channel constants read once, output written once; a whole network's
    intermediate activations need not leave the chip and are not counted."""
    if case["kind"] == "net":
        net = _net_spec(case)
        io = net.B * (net.Cin * net.Tin + net.Cout * net.Tout) * (4 if case["entry"] == "f32" else 1)
        consts = sum(o.Cout * (12 if o.has_bias else 8) for o in net.ops)
        return {"bytes": io + W.net_weight_count(net) + consts, "flops": 2 * W.net_macs(net)}
    if case["kind"] == "layer":
        B, Cin, Cout, T, k = (case[n] for n in ("B", "Cin", "Cout", "T", "k"))
        fan = k if case["layer"] == "dw" else Cin * k
        return {"bytes": B * T * (Cin + Cout * (2 if case["res"] else 1)) + Cout * (fan + 12), "flops": 2 * B * T * Cout * fan}
    if case["kind"] == "softmax":
        n = case["rows"] * case["L"]
        return {"bytes": 5 * n, "flops": 10 * n}
    n, nw = case["B"] * case["C"] * case["T"], case["Cout"] * case["C"] * case["k"]
    return {"bytes": 4 * n + 5 * nw + 32 * case["Cout"], "flops": 2 * n + 4 * nw}


def tolerance(case):
    return "exact"          # integers everywhere; the few floats are single operations, rounded once
