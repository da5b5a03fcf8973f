"""Workloads of the token shuffle as a program that uses it runs them: what an MoE layer asks of the library per
call, from a handful of decode tokens to a long prefill batch, both directions of the path (out to the experts and
back), all payload types, and the descriptor engine on its own.

A case is a dict of plain values.  `prepare` makes what the program holds before the call (inputs, layout, output
tensors), `run` is one pass through the public entry points, `exact` the same result from plain torch in 64 bits.

kinds
  decode     fusco_plan_dispatch + fusco_combine: a decode batch of one planner tile
  step       fusco_plan + fusco_dispatch + fusco_combine: the shuffle of one MoE layer of a prefill batch; the
             experts' output is a tensor of its own, since the expert computation sits between the two calls
  train      a step followed by its gradients: the output's gradient is dispatched to the experts' rows, and the
             gradient of the expert inputs is brought back to the tokens (a combine whose weights are 1)
  two_level  plan, dispatch that also writes the deduplicated per-device tensors, two-hop combine: the form in which
             rows or partial sums go over links between devices
  plan       fusco_plan alone, for programs that plan a batch once and move several tensors by the same plan
  segments   scan of a descriptor list, pack into slices for a network engine, unpack of the packed stream to other
             places: segments of any size, as for key-value blocks or ragged rows
"""
import math

import torch

import paper_2512_22036_amd as fusco

_PAYLOAD = {"bf16": (torch.bfloat16, 2), "f32": (torch.float32, 4), "fp8": (torch.uint8, 1)}
_SLICE = 1 << 20


def listed():
    return [
        # a few sequences being decoded, fp8 rows with one fp32 scale per 128 elements: launches and latency only
        dict(name="decode_4", kind="decode", N=4, H=7168, k=8, E=256, D=64, payload="fp8", out="bf16", routing="normal"),
        # the decode batch of the benchmark configurations
        dict(name="decode_fp8", kind="decode", N=128, H=7168, k=8, E=256, D=64, payload="fp8", out="bf16", routing="normal"),
        # the smallest of the benchmark configurations: cache resident, bound by the chain of launches
        dict(name="tiny_step", kind="step", N=4096, H=1024, k=2, E=16, D=4, payload="bf16", out="bf16", routing="normal"),
        # a ragged chunk of a chunked prefill: nothing is a power of two, fp32 output for the residual stream
        dict(name="ragged_step", kind="step", N=1537, H=2880, k=6, E=160, D=5, payload="bf16", out="f32", routing="normal"),
        # the benchmark configurations of large batches
        dict(name="qwen3_step", kind="step", N=16384, H=4096, k=8, E=128, D=16, payload="bf16", out="bf16", routing="normal"),
        dict(name="dsv3_step", kind="step", N=8192, H=7168, k=8, E=256, D=8, payload="bf16", out="bf16", routing="normal"),
        # popular experts, each token's experts on at most four devices: a long prefill batch
        dict(name="skewed_step", kind="step", N=32768, H=7168, k=8, E=256, D=8, payload="bf16", out="bf16", routing="zipf"),
        # the benchmark batch with fp8 rows and their scales on the way out, bf16 rows on the way back
        dict(name="fp8_prefill", kind="step", N=8192, H=7168, k=8, E=256, D=8, payload="fp8", out="bf16", routing="normal"),
        # fp32 training: rows out and back, then their gradients
        dict(name="train_f32", kind="train", N=8192, H=2048, k=4, E=64, D=8, payload="f32", out="f32", routing="normal"),
        # both levels of the plan written out, for links between devices
        dict(name="two_level", kind="two_level", N=4096, H=7168, k=8, E=256, D=8, payload="bf16", out="bf16", routing="normal"),
        # a plan for a batch that is moved tensor by tensor
        dict(name="plan_131072", kind="plan", N=131072, H=0, k=8, E=256, D=8, payload="bf16", out="bf16", routing="normal"),
        # ragged segments of 16 bytes to 14 KiB, about 290 MB, sent in slices and received
        dict(name="segments", kind="segments", n=40000, top=14336),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "step", "step", "step", "step", "train", "two_level", "plan", "segments"])
    if kind == "segments":
        top = 16 * _log_uniform(rng, 64, 2048)
        return dict(kind=kind, n=_log_uniform(rng, 500, max(501, min(200000, 1_200_000_000 // top))), top=top)
    E, D = rng.choice([(16, 4), (32, 8), (60, 4), (64, 8), (128, 16), (160, 5), (256, 8), (256, 64), (384, 8)])
    k = rng.choice([1, 2, 4, 4, 6, 8, 8, 8, 10])
    payload = rng.choice(["bf16", "bf16", "fp8"]) if kind in ("decode", "step") else ("f32" if kind == "train" else "bf16")
    H = 512 * rng.randint(2, 16) if payload == "fp8" else 8 * rng.randint(64, 1024)
    out = "f32" if payload == "f32" else rng.choice(["bf16", "bf16", "f32"])
    routing = "normal" if kind == "two_level" else rng.choice(["normal", "normal", "zipf"])
    lo, hi = {"decode": (1, 2048 // k), "plan": (2048, 262144)}.get(kind, (256, 32768))
    case = dict(kind=kind, N=_log_uniform(rng, lo, hi), H=H, k=k, E=E, D=D, payload=payload, out=out, routing=routing)
    if kind == "plan":
        return dict(case, H=0, payload="bf16", out="bf16")
    while work(case)["bytes"] > 6e9:
        case["N"] = case["N"] * 2 // 3
    return case


def _routing(case, gen):
    """Router output: the k experts of every token in descending score, and their weights (softmax over the chosen)."""
    N, E, k, D = case["N"], case["E"], case["k"], case["D"]
    if case["routing"] == "zipf":
        rank = torch.randperm(E, generator=gen, device="cuda") + 1
        noise = torch.rand((N, E), generator=gen, device="cuda").clamp_(1e-7, 1 - 1e-7)
        score = -1.2 * torch.log(rank.float()) - torch.log(-torch.log(noise))
        keep = min(4, D)
        if keep < D and keep * (E // D) >= k:   # device-limited routing
            best = score.view(N, D, E // D).amax(dim=2).topk(keep, dim=1).indices
            allowed = torch.zeros((N, D), dtype=torch.bool, device="cuda").scatter_(1, best, True)
            score = score.masked_fill(~allowed.repeat_interleave(E // D, dim=1), -math.inf)
    else:
        score = torch.randn((N, E), generator=gen, device="cuda")
    top = score.topk(k, dim=1)
    return top.indices.to(torch.int32).contiguous(), torch.softmax(top.values, dim=1).contiguous()


def _rows(n, H, payload, gen):
    if payload == "fp8":   # e4m3 bytes of normal values: sign, exponents around 1, any mantissa
        return torch.randint(0, 0x7F, (n, H), generator=gen, device="cuda", dtype=torch.uint8)
    return torch.randn((n, H), generator=gen, device="cuda", dtype=_PAYLOAD[payload][0])


def _empty(rows, H, payload):
    return torch.empty((rows, H), dtype=_PAYLOAD[payload][0], device="cuda")


_ARRAYS = ("exp_count", "exp_off", "send_count", "send_off", "pair_slot", "slot_pair", "slot_token", "send_src",
           "pair_send_row", "slot_send_row", "pair_first", "status", "tile_slots")


def _stream_bytes(case):
    n, units = case["n"], case["top"] // 16
    return 16 * (n + sum(i * units // n for i in range(n)))


def _inputs(case, seed):
    """The inputs alone, from the seed: shared by prepare and exact."""
    gen = torch.Generator(device="cuda").manual_seed(seed * 7919 + 17)
    if case["kind"] == "segments":
        n, units = case["n"], case["top"] // 16
        size = 16 * (1 + torch.arange(n, device="cuda") * units // n)   # every size up to top, as often as the others
        size = size[torch.randperm(n, generator=gen, device="cuda")]
        ends = []
        for _ in range(2):   # the segments lie in another order in the sender's and in the receiver's memory
            order = torch.randperm(n, generator=gen, device="cuda")
            off = torch.empty_like(size)
            off[order] = torch.cumsum(size[order], 0) - size[order]
            ends.append(torch.stack([off, size], dim=1).contiguous())
        total = _stream_bytes(case)
        src = torch.randint(0, 256, (total,), generator=gen, device="cuda", dtype=torch.uint8)
        return dict(src=src, src_desc=ends[0], dst_desc=ends[1], total=total)
    A, w = _routing(case, gen)
    got = dict(A=A, w=w)
    if case["kind"] == "plan":
        return got
    N, H, P, payload = case["N"], case["H"], case["N"] * case["k"], case["payload"]
    got["x"] = _rows(N, H, payload, gen)
    if payload == "fp8":
        got["scales"] = torch.rand((N, H // 128), generator=gen, device="cuda") * 0.01 + 0.001
    got["y"] = _rows(P, H, "f32" if payload == "f32" else "bf16", gen)
    if case["kind"] == "train":
        got["grad_out"] = _rows(N, H, payload, gen)
        got["grad_rows"] = _rows(P, H, payload, gen)
        got["ones"] = torch.ones_like(w)
    return got


def prepare(case, seed):
    s = _inputs(case, seed)
    s["kind"] = case["kind"]
    if case["kind"] == "segments":
        n, total = case["n"], s["total"]
        s["capacity"] = -(-total // _SLICE) * _SLICE
        s["cum"] = torch.zeros((n + 1,), dtype=torch.int64, device="cuda")
        s["status"] = torch.zeros((1,), dtype=torch.int32, device="cuda")
        s["fill"] = torch.zeros((s["capacity"] // _SLICE,), dtype=torch.int32, device="cuda")
        s["packed"] = torch.zeros((s["capacity"],), dtype=torch.uint8, device="cuda")
        s["dst"] = torch.zeros((total,), dtype=torch.uint8, device="cuda")
        s["outputs"] = [s["cum"], s["status"], s["fill"], s["packed"], s["dst"]]
        return s
    N, H, k, P, payload = case["N"], case["H"], case["k"], case["N"] * case["k"], case["payload"]
    L = s["layout"] = fusco.Layout(N, k, case["E"], case["D"])
    L.mem.zero_()   # send rows beyond the last one in use are never written
    outputs = [L.array(name) for name in _ARRAYS]
    if case["kind"] != "plan":
        s["rows"] = _empty(P, H, payload)
        s["out"] = _empty(N, H, case["out"])
        s["planes"] = {}
        outputs += [s["rows"], s["out"]]
        if payload == "fp8":
            s["planes"] = dict(x_aux=s["scales"], expert_aux=_empty(P, H // 128, "f32"))
            outputs.append(s["planes"]["expert_aux"])
    if case["kind"] == "train":
        s["grad_y"], s["grad_x"] = _empty(P, H, payload), _empty(N, H, payload)
        outputs += [s["grad_y"], s["grad_x"]]
    if case["kind"] == "two_level":
        s["wire"] = torch.zeros((L.send_cap, H), dtype=_PAYLOAD[payload][0], device="cuda")
        s["partial"] = torch.zeros((L.send_cap, H), dtype=torch.float32, device="cuda")
        outputs += [s["wire"], s["partial"]]
    s["outputs"] = outputs
    return s


def run(s):
    kind = s["kind"]
    if kind == "segments":
        fusco.fusco_segments_scan(s["src_desc"], s["cum"], s["status"])
        fusco.fusco_segments_copy(s["src"], s["src_desc"], s["packed"], None, s["cum"], s["capacity"], s["status"],
                                  slice_bytes=_SLICE, slice_fill=s["fill"])
        fusco.fusco_segments_copy(s["packed"], None, s["dst"], s["dst_desc"], s["cum"], s["capacity"], s["status"])
        return s["outputs"]
    L = s["layout"]
    if kind == "decode":
        fusco.fusco_plan_dispatch(L, s["A"], s["x"], s["rows"], **s["planes"])
        fusco.fusco_combine(L, s["y"], s["w"], s["out"])
        return s["outputs"]
    fusco.fusco_plan(L, s["A"])
    if kind == "plan":
        return s["outputs"]
    if kind == "two_level":
        fusco.fusco_dispatch(L, s["x"], s["rows"], send_buf=s["wire"], flags=fusco.DISPATCH_EXPERT | fusco.DISPATCH_WIRE)
        fusco.fusco_combine_two_hop(L, s["y"], s["w"], s["partial"], s["out"])
        return s["outputs"]
    fusco.fusco_dispatch(L, s["x"], s["rows"], **s["planes"])
    fusco.fusco_combine(L, s["y"], s["w"], s["out"])
    if kind == "train":
        fusco.fusco_dispatch(L, s["grad_out"], s["grad_y"])
        fusco.fusco_combine(L, s["grad_rows"], s["ones"], s["grad_x"])
    return s["outputs"]


def _send_rows(case):
    """Expected number of (token, device) pairs under the uniform routing."""
    E, D, k = case["E"], case["D"], case["k"]
    miss = 1.0
    for i in range(k):
        miss *= max(0, E - E // D - i) / (E - i)
    return case["N"] * D * (1.0 - miss)


def work(case):
    if case["kind"] == "segments":
        n, total = case["n"], _stream_bytes(case)
        return {"bytes": 4 * total + n * 16 * 2 + 8 * (n + 1), "flops": 0}
    N, H, k = case["N"], case["H"], case["k"]
    P = N * k
    plan = 4 * P + 29 * P   # the routing in, the descriptor arrays out
    if case["kind"] == "plan":
        return {"bytes": plan, "flops": 0}
    row = H + H // 128 * 4 if case["payload"] == "fp8" else H * _PAYLOAD[case["payload"]][1]
    y_row, out_row = (4 * H if case["payload"] == "f32" else 2 * H), H * _PAYLOAD[case["out"]][1]
    one = (N + P) * row + P * y_row + N * out_row + 4 * P
    if case["kind"] == "train":
        return {"bytes": plan + 2 * one, "flops": 4 * P * H}
    if case["kind"] == "two_level":
        one += int(_send_rows(case)) * (row + 4 * H)
    return {"bytes": plan + one, "flops": 2 * P * H}


def tolerance(case):
    # Bytes and whole numbers are moved, and the weighted sums have a stated order: fp32 fused multiply-adds in
    # ascending entry, one rounding at the end.  Two implementations of that agree bit for bit.
    return "exact"


def exact(case, seed):
    if case["kind"] in ("plan", "segments"):
        return None   # whole numbers and bytes
    s = _inputs(case, seed)
    N, H, k, E, D = case["N"], case["H"], case["k"], case["E"], case["D"]
    A = s["A"].long()
    order = torch.argsort(A.flatten(), stable=True)   # slot -> pair: expert by expert, tokens ascending
    slot = torch.empty_like(order)
    slot[order] = torch.arange(N * k, device="cuda")
    slot, token = slot.view(N, k), order // k

    def combine(y, w):
        out = torch.empty((N, H), dtype=torch.float64, device="cuda")
        for t in range(0, N, 1024):
            acc = torch.zeros((min(1024, N - t), H), dtype=torch.float64, device="cuda")
            for j in range(k):
                acc += w[t:t + 1024, j:j + 1].double() * y[slot[t:t + 1024, j]].double()
            out[t:t + 1024] = acc
        return out

    out = combine(s["y"], s["w"])
    got = [None] * len(_ARRAYS)
    if case["payload"] == "fp8":
        return got + [None, out, s["scales"][token]]
    got += [s["x"][token], out]
    if case["kind"] == "train":
        got += [s["grad_out"][token], combine(s["grad_rows"], s["ones"])]
    if case["kind"] == "two_level":
        dev = A // (E // D)
        has = torch.zeros((N, D), dtype=torch.bool, device="cuda").scatter_(1, dev, True)
        where = has.t().nonzero()   # (device, token) of every send row, device-major
        row_of = torch.full((N, D), -1, dtype=torch.int64, device="cuda")
        row_of[where[:, 1], where[:, 0]] = torch.arange(where.shape[0], device="cuda")
        cap = N * min(k, D)
        wire = torch.zeros((cap, H), dtype=s["x"].dtype, device="cuda")
        wire[:where.shape[0]] = s["x"][where[:, 1]]
        partial = torch.zeros((cap, H), dtype=torch.float64, device="cuda")
        for j in range(k):
            for t in range(0, N, 1024):
                at = row_of[torch.arange(t, min(t + 1024, N), device="cuda"), dev[t:t + 1024, j]]
                partial[at] += s["w"][t:t + 1024, j:j + 1].double() * s["y"][slot[t:t + 1024, j]].double()
        got += [wire, partial]
    return got
