"""The calls that a program using this library makes, with the sizes it makes them at.

A serving program quantizes the visual tokens of new sequences (prefill), then, for every token it
generates and every layer, appends the new key and value to the 16-bit tail and attends; the
calibration parameters are searched once per model.  Shapes are those of the benchmark's workloads
(`paper_2502_14882_amd.synth.WORKLOADS`) and of the tests, from one short row to a full prefill.

A case is a dict of plain values:
    kind        "decode" (one attention call), "step" (the append + attend of `layers` layers
                recorded into one HIP graph, lengths on the device, replayed), "quantize", "tau"
    batch, n_q_heads, n_kv_heads, head_dim, n_vis, n_text, bits
    k_group, v_axis, v_group    keys are quantized per channel over k_group tokens; values per token
                (v_axis 1, channels per group) or per channel (v_axis 0, tokens per group)
    calib       "dynamic", "none" or "fixed", with tau1, tau2
    dist        distribution of the keys: "uniform", "student_t", "fixed" or "none" (outlier channels)
"""
from __future__ import annotations

import math

import torch

from paper_2502_14882_amd import binding as cq
from paper_2502_14882_amd import synth

CHANNEL, TOKEN = 0, 1
TAUS = (0.0, 1.0, 2.0, 3.0)
FIXED_RANGE = (-12.0, 12.0)      # gamma, delta of a calibration with given bounds


def _case(kind, batch, n_q_heads, n_kv_heads, n_vis, n_text, bits, head_dim=128, k_group=128,
          v_axis=TOKEN, v_group=None, calib="dynamic", tau1=1, tau2=2, dist="uniform", layers=1):
    return dict(kind=kind, batch=batch, n_q_heads=n_q_heads, n_kv_heads=n_kv_heads,
                head_dim=head_dim, n_vis=n_vis, n_text=n_text, bits=bits, k_group=k_group,
                v_axis=v_axis, v_group=head_dim if v_group is None else v_group, calib=calib,
                tau1=tau1, tau2=tau2, dist=dist, layers=layers)


def listed():
    def c(name, *a, **kw):
        return dict(_case(*a, **kw), name=name)

    return [
        # one head over a thousand tokens: nothing but the cost of a call
        c("decode_tiny", "decode", 1, 1, 1, 1024, 32, 1, dist="fixed"),
        # interactive use, one sequence: eight layers of an 8B-shaped model per recorded step
        c("step_single", "step", 1, 32, 8, 3328, 128, 1, layers=8),
        # the same layers for a batch of sixteen sequences
        c("step_batch", "step", 16, 32, 8, 3328, 128, 1, layers=4),
        # multi-frame video, the largest batch of the benchmark's decode workloads
        c("decode_video", "decode", 64, 32, 8, 8192, 512, 1),
        # long context, six query heads per KV head, heavy-tailed key channels
        c("decode_long", "decode", 8, 48, 8, 65536, 1024, 1, dist="student_t"),
        # a user who trades memory for accuracy: 4-bit codes, keys in groups of 64 tokens
        c("decode_wide", "decode", 16, 32, 8, 3328, 128, 4, k_group=64),
        # the paper's own scheme (one pair per channel over the whole sequence, keys and values) on
        # an image whose token count is not a round number, 2 bits
        c("decode_whole", "decode", 8, 32, 8, 3003, 77, 2, k_group=3003, v_axis=CHANNEL,
          v_group=3003),
        # a small model's heads of 64 channels
        c("decode_head64", "decode", 16, 16, 4, 3328, 100, 1, head_dim=64, k_group=64),
        # prefill of a large batch (keys and values), and of one sequence
        c("quantize_prefill", "quantize", 128, 8, 8, 16384, 0, 1),
        c("quantize_single", "quantize", 1, 8, 8, 3328, 0, 2),
        # prefill under the paper's own scheme, ragged token count
        c("quantize_whole", "quantize", 8, 8, 8, 3003, 0, 2, k_group=3003, v_axis=CHANNEL,
          v_group=3003),
        # the 4 x 4 grid of calibration parameters on a calibration batch
        c("tau_search", "tau", 4, 32, 8, 3328, 128, 1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(("decode", "step", "quantize", "tau"), (55, 15, 20, 10))[0]
    head_dim = rng.choices((128, 64, 256), (80, 15, 5))[0]
    n_q, n_kv = rng.choice(((1, 1), (4, 4), (8, 2), (14, 2), (16, 4), (16, 8), (24, 8), (32, 8),
                            (48, 8), (64, 8), (16, 16)))
    bits = rng.choices((1, 2, 4, 8), (45, 30, 15, 10))[0]
    if rng.random() < 0.25:                  # statistics over the whole sequence, any token count
        n_vis = _log(rng, 200, 16384)
        k_group, v_axis, v_group = n_vis, CHANNEL, n_vis
        if rng.random() < 0.4:
            v_axis, v_group = TOKEN, head_dim
    else:
        k_group = rng.choice((32, 64, 128, 128, 128))
        v_axis, v_group, unit = TOKEN, head_dim, k_group
        if rng.random() < 0.2:
            v_axis, v_group = CHANNEL, rng.choice((64, 128))
            unit = max(unit, v_group)
        n_vis = max(1, _log(rng, 256, 65536) // unit) * unit
    # as many sequences as a layer of the video workload holds tokens; a quarter for the search
    tokens = (1 << 20) if kind == "tau" else 64 * 8 * 8192
    batch = _log(rng, 1, max(1, min(64, tokens // (n_kv * n_vis))))
    n_text = 0 if kind == "quantize" else _log(rng, 1, 1024)
    layers = 1
    if kind == "step":
        layers = max(1, min(8, tokens // (batch * n_kv * n_vis)))
    calib = rng.choices(("dynamic", "none", "fixed"), (70, 20, 10))[0]
    return _case(kind, batch, n_q, n_kv, n_vis, n_text, bits, head_dim=head_dim, k_group=k_group,
                 v_axis=v_axis, v_group=v_group, calib=calib, tau1=rng.randrange(4),
                 tau2=rng.randrange(4), dist=rng.choice(("uniform", "uniform", "student_t", "none")),
                 layers=layers)


def _seed_of(seed, layer):
    return 100003 * int(seed) + 17 * layer + 5


def _inputs(case, seed, layer=0):
    """fp16 tensors of one layer: k, v, q, and a tail with room for one more token."""
    w = synth.Workload(case["kind"], 0, case["batch"], case["n_q_heads"], case["n_kv_heads"],
                       case["head_dim"], case["n_vis"], case["n_text"] + 1, case["dist"])
    parts = ("k", "v") if case["kind"] == "quantize" else ("k", "v", "q", "k_text", "v_text")
    return synth.make_inputs(w, "cuda", _seed_of(seed, layer), parts)


def _layout(case):
    return cq.make_layout(case["batch"], case["n_q_heads"], case["n_kv_heads"], case["head_dim"],
                          case["n_vis"], case["bits"], CHANNEL, case["v_axis"], case["k_group"],
                          case["v_group"])


def _calib(case):
    mode = {"none": cq.CQ_CALIB_NONE, "dynamic": cq.CQ_CALIB_DYNAMIC,
            "fixed": cq.CQ_CALIB_FIXED}[case["calib"]]
    return cq.make_calib(mode, case["tau1"], case["tau2"], *FIXED_RANGE)


def _workspace(n_bytes):
    return torch.empty(max(n_bytes, 256), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    lay = _layout(case)
    kind = case["kind"]
    st = {"kind": kind, "lay": lay}
    if kind == "quantize":
        x = _inputs(case, seed)
        st.update(k=x["k"], v=x["v"],
                  k_out=cq.alloc_qtensor(lay, CHANNEL, case["k_group"], "cuda"),
                  v_out=cq.alloc_qtensor(lay, case["v_axis"], case["v_group"], "cuda"))
        return st
    st["n_text"] = n_text = case["n_text"]
    if kind == "tau":
        x = _inputs(case, seed)
        k, _ = cq.cq_quantize_kv(lay, x["k"], x["v"])
        ws = _workspace(cq.cq_tau_search_workspace_bytes(lay, n_text, len(TAUS), len(TAUS)))
        st.update(q=x["q"], k_exact=x["k"], k=k, k_text=x["k_text"], ws=ws)
        return st
    st["calib"] = calib = _calib(case)
    if kind == "decode":
        x = _inputs(case, seed)
        k, v = cq.cq_quantize_kv(lay, x["k"], x["v"])
        st.update(q=x["q"], k=k, v=v, k_text=x["k_text"], v_text=x["v_text"],
                  out=torch.empty_like(x["q"]),
                  ws=_workspace(cq.cq_decode_workspace_bytes(lay, n_text, calib)))
        return st
    # A recorded step: every layer appends its new token to its tail and attends; the lengths live
    # on the device.  The step begins by setting them back, so that a replay attends to the same
    # tokens again.
    cap = n_text + 1
    ws = _workspace(cq.cq_decode_workspace_bytes(lay, cap, calib))
    lengths = torch.full((case["layers"],), n_text, dtype=torch.int32, device="cuda")
    layers = []
    for i in range(case["layers"]):
        x = _inputs(case, seed, i)
        k, v = cq.cq_quantize_kv(lay, x.pop("k"), x.pop("v"))
        new = [x[t][:, :, n_text:].contiguous() for t in ("k_text", "v_text")]
        for t in ("k_text", "v_text"):
            x[t][:, :, n_text:] = 0
        layers.append(dict(q=x["q"], k=k, v=v, k_text=x["k_text"], v_text=x["v_text"],
                           k_new=new[0], v_new=new[1], length=lengths[i:i + 1],
                           out=torch.empty_like(x["q"])))

    def step():
        lengths.fill_(n_text)
        for y in layers:
            cq.cq_append_text_kv_devlen(lay, y["k_text"], y["v_text"], y["length"], y["k_new"],
                                        y["v_new"])
            cq.cq_decode_attn_devlen(lay, y["q"], y["k"], y["v"], y["k_text"], y["v_text"],
                                     y["length"], cap, calib, out=y["out"], workspace=ws)

    step()                                   # once outside the recording, as first calls go
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    st.update(graph=graph, layers=layers, lengths=lengths, ws=ws)
    return st


def run(state):
    kind, lay = state["kind"], state["lay"]
    if kind == "decode":
        return cq.cq_decode_attn(lay, state["q"], state["k"], state["v"], state["k_text"],
                                 state["v_text"], state["n_text"], state["calib"],
                                 out=state["out"], workspace=state["ws"])
    if kind == "step":
        state["graph"].replay()
        return {"out": [y["out"] for y in state["layers"]],
                "k_text": [y["k_text"] for y in state["layers"]],
                "v_text": [y["v_text"] for y in state["layers"]], "lengths": state["lengths"]}
    if kind == "quantize":
        k, v = cq.cq_quantize_kv(lay, state["k"], state["v"], state["k_out"], state["v_out"])
        return {"k": list(k), "v": list(v)}
    return cq.cq_tau_search(lay, state["q"], state["k_exact"], state["k"], state["k_text"],
                            state["n_text"], TAUS, TAUS, workspace=state["ws"])


def work(case):
    B, Hq, Hkv, d = (case[n] for n in ("batch", "n_q_heads", "n_kv_heads", "head_dim"))
    n, t, b = case["n_vis"], case["n_text"], case["bits"]
    rows = B * Hkv
    codes = rows * n * d * b // 8
    k_par = rows * (n // case["k_group"]) * d * 6
    v_par = 6 * (rows * (n // case["v_group"]) * d if case["v_axis"] == CHANNEL
                 else rows * n * (d // case["v_group"]))
    if case["kind"] == "quantize":
        # per element: two comparisons for the extrema, the code by subtract, multiply, round
        return {"bytes": 2 * rows * n * d * 2 + 2 * codes + k_par + v_par,
                "flops": 2 * rows * n * d * 5}
    if case["kind"] == "tau":
        return {"bytes": rows * n * d * 2 + codes + k_par + rows * t * d * 2 + B * Hq * d * 2
                + 8 * len(TAUS) ** 2,
                "flops": 2 * B * Hq * d * (2 * n + t)}
    t += case["kind"] == "step"
    one = 2 * codes + k_par + v_par + rows * t * d * 4 + 2 * B * Hq * d * 2
    if case["kind"] == "step":
        one += rows * d * 8                  # the new key and value, read and written
    return {"bytes": case["layers"] * one, "flops": case["layers"] * 4 * B * Hq * d * (n + t)}


def tolerance(case):
    if case["kind"] == "quantize":
        return "exact"
    if case["kind"] == "tau":
        # 32-bit logits, everything after them in 64: up to 5e-6 from 64 bits where one key stands out
        return {"rel": 2e-5, "max": 2e-4}
    return {"rel": 1e-3, "max": 1e-2}        # results in fp16: 1.5e-4 to 2.4e-4 from 64 bits


# ---- the same in 64 bits, from the definitions

def _quantized(x, axis, group, bits):
    """Codes (float64), scale (float32) and minimum (fp16) of x [H, n, d] in 64 bits, and the
    dequantized tensor."""
    H, n, d = x.shape
    x = x.double()
    g = x.view(H, n // group, group, d) if axis == CHANNEL else x.view(H, n, d // group, group)
    dim = 2 if axis == CHANNEL else 3
    lo, hi = g.amin(dim, keepdim=True), g.amax(dim, keepdim=True)
    top, width = float((1 << bits) - 1), hi - lo
    codes = torch.where(width > 0, torch.round((g - lo) * top / width.clamp_min(1e-300)), 0.0)
    scale, low = (width / top).float(), lo.half() + 0.0
    deq = codes * scale.double() + lo
    return codes.view(H, n, d), scale.squeeze(dim), low.squeeze(dim), deq.view(H, n, d)


def _packed(codes, bits):
    per = 32 // bits
    c = codes.to(torch.int64).view(*codes.shape[:-1], -1, per)
    at = torch.tensor([32 - bits * (1 + i) for i in range(per)], device=codes.device)
    words = (c << at).sum(-1)
    return torch.where(words >= 1 << 31, words - (1 << 32), words).to(torch.int32)


def _calibrated(case, s):
    """g of the visual logits s [.., n]."""
    if case["calib"] == "none":
        return s
    lo, hi = s.amin(-1, keepdim=True), s.amax(-1, keepdim=True)
    if case["calib"] == "fixed":
        lo, hi = torch.full_like(lo, FIXED_RANGE[0]), torch.full_like(hi, FIXED_RANGE[1])
    return _line(s, lo, hi, case["tau1"], case["tau2"])


def _line(s, lo, hi, tau1, tau2):
    width = hi - lo
    slope = torch.where(width == 0, 1.0, (width + tau1 - tau2) / width)
    return slope * (s - lo) + lo - tau1


def _logits(q, k):
    """q [Hkv, g, d] . k [Hkv, n, d], scaled."""
    return torch.matmul(q, k.transpose(1, 2).contiguous()) / math.sqrt(q.shape[-1])


def _attend(case, x, b, n_text):
    """One sequence's decode step in 64 bits: [Hq, d]."""
    Hkv, d = case["n_kv_heads"], case["head_dim"]
    kd = _quantized(x["k"][b], CHANNEL, case["k_group"], case["bits"])[3]
    vd = _quantized(x["v"][b], case["v_axis"], case["v_group"], case["bits"])[3]
    q = x["q"][b].double().view(Hkv, -1, d)
    kt, vt = x["k_text"][b, :, :n_text].double(), x["v_text"][b, :, :n_text].double()
    s = torch.cat([_calibrated(case, _logits(q, kd)), _logits(q, kt)], -1)
    p = torch.softmax(s, -1)
    n = case["n_vis"]
    o = torch.matmul(p[..., :n].contiguous(), vd) + torch.matmul(p[..., n:].contiguous(), vt)
    return o.view(-1, d)


def _tau_grid(case, x):
    Hkv, d, n = case["n_kv_heads"], case["head_dim"], case["n_vis"]
    total, t = 0.0, case["n_text"]
    for b in range(case["batch"]):
        q = x["q"][b].double().view(Hkv, -1, d)
        text = _logits(q, x["k_text"][b, :, :t].double())
        ref = torch.softmax(torch.cat([_logits(q, x["k"][b].double()), text], -1), -1)
        s = _logits(q, _quantized(x["k"][b], CHANNEL, case["k_group"], case["bits"])[3])
        lo, hi = s.amin(-1, keepdim=True), s.amax(-1, keepdim=True)
        grid = [[((torch.softmax(torch.cat([_line(s, lo, hi, t1, t2), text], -1), -1) - ref) ** 2)
                 .mean(-1).sum() for t2 in TAUS] for t1 in TAUS]
        total = total + torch.stack([torch.stack(r) for r in grid])
    return total / (case["batch"] * case["n_q_heads"])


def exact(case, seed):
    kind, B, n_text = case["kind"], case["batch"], case["n_text"]
    if kind == "quantize":
        x = _inputs(case, seed)
        res = {}
        for name, axis, group in (("k", CHANNEL, case["k_group"]),
                                  ("v", case["v_axis"], case["v_group"])):
            rows = []
            for b in range(B):
                codes, scale, low, _ = _quantized(x[name][b], axis, group, case["bits"])
                rows.append((_packed(codes, case["bits"]), scale, low))
            res[name] = [torch.stack(t) for t in zip(*rows)]
        return res
    if kind == "tau":
        return _tau_grid(case, _inputs(case, seed))
    if kind == "decode":
        x = _inputs(case, seed)
        return torch.stack([_attend(case, x, b, n_text) for b in range(B)])
    res = {"out": [], "k_text": [], "v_text": [],
           "lengths": torch.full((case["layers"],), n_text + 1, dtype=torch.int32)}
    for i in range(case["layers"]):
        x = _inputs(case, seed, i)
        res["out"].append(torch.stack([_attend(case, x, b, n_text + 1) for b in range(B)]))
        res["k_text"].append(x["k_text"])
        res["v_text"].append(x["v_text"])
    return res
