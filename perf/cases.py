"""The workloads whose time is measured: what a program that uses the layer has it do.

Four kinds of pass, each through the calls that such a program makes:

  fwd     one layer of a prefill: l2a_route_compact + l2a_attn_fwd
  train   one layer of a training step: l2a_route_compact + l2a_attn_fwd + l2a_attn_bwd
  decode  one token per sequence against the KV caches: l2a_attn_decode
  router  the router's decision for every token: l2a_router_decide

Head layouts, windows, routed fractions and mask kinds are those of the workloads in
paper_2603_17484_amd/inputs.py; lengths run from one short prompt to 128K tokens.  The tensors are
N(0,1), the masks Bernoulli or bursty, as everywhere in this repository.
"""
import ctypes
import math

import torch

from paper_2603_17484_amd import binding as B
from paper_2603_17484_amd import inputs as gen
from paper_2603_17484_amd.runner import Layer

DEV = "cuda"


# --------------------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------------------
def layer_case(kind, name=None, **kw):
    """kind: fwd or train.  heads: query heads, kv: KV heads, mask_heads: 1 (a decision per token, what the
    router emits) or one per query head; burst: mean run of routed tokens, 0 for independent tokens;
    separate: Local and Global modules with projections of their own."""
    case = {"kind": kind, "B": 1, "T": 4096, "heads": 28, "kv": 4, "D": 128, "W": 4096, "dtype": "bf16",
            "mask_heads": 1, "f": 0.2, "burst": 0, "separate": False}
    case.update(kw)
    if name:
        case["name"] = name
    return case


def decode_case(name=None, **kw):
    """capacity: tokens a sequence's cache holds; routed: how many of the B sequences route their new token;
    separate: Local module with a ring cache of its own, Global module with the full cache (two calls)."""
    case = {"kind": "decode", "B": 8, "capacity": 131072, "heads": 28, "kv": 4, "W": 4096, "routed": 2,
            "separate": False}
    case.update(kw)
    if name:
        case["name"] = name
    return case


def router_case(name=None, **kw):
    case = {"kind": "router", "B": 1, "T": 32768, "C": 3584, "dtype": "bf16"}
    case.update(kw)
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # one conversation being generated, its token routed to Global attention: latency of a single step
        decode_case("decode_1x32k", B=1, capacity=32768, routed=1),
        # a long-context serving batch, one token in four routed
        decode_case("decode_8x128k", B=8, capacity=131072, routed=2),
        # a wide serving batch of the model with separate Local and Global modules (Hq = 32, Hkv = 8)
        decode_case("decode_32x16k_separate", B=32, capacity=16384, heads=32, kv=8, routed=8, separate=True),
        # the router over a prefill's hidden states (3584 channels: 28 heads x 128)
        router_case("router_32k"),
        # a short prompt of odd length: launches and latency count
        layer_case("fwd", "fwd_1k", T=1001),
        # an ordinary prompt
        layer_case("fwd", "fwd_4k", T=4096),
        # a long prompt (the 32K forward configuration)
        layer_case("fwd", "fwd_32k", T=32768),
        # fine-tuning on ordinary lengths: two sequences, separate modules, the router's task-loss gradient wanted
        layer_case("train", "train_2x4k_separate", B=2, T=4000, separate=True),
        # long-context training, Hq = 32 / Hkv = 8, a bursty mask per head, odd length
        layer_case("train", "train_16k_bursty", T=16379, heads=32, kv=8, mask_heads=32, burst=32),
        # the headline: 128K tokens, a Bernoulli mask per head, 80 % of the tokens skip Global attention
        layer_case("train", "train_128k", T=131072, mask_heads=28),
        # the small 32-bit configuration that checks of a model's numerics run on
        layer_case("train", "train_2k_fp32", T=2048, heads=1, kv=1, D=64, W=256, dtype="fp32"),
        # a 32-bit layer with grouped heads of 128 channels
        layer_case("train", "train_4k_fp32", T=4096, heads=8, kv=2, W=1024, dtype="fp32"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "router", "fwd", "fwd", "train", "train", "fp32"])
    heads, kv = rng.choice([(28, 4), (32, 8)])
    if kind == "decode":
        batch = _log_int(rng, 1, 64)
        capacity = _log_int(rng, 1024, min(131072, 2 ** 20 // batch))
        return decode_case(B=batch, capacity=capacity, heads=heads, kv=kv, W=rng.choice([1024, 4096]),
                           routed=rng.randint(0, batch), separate=rng.random() < 0.4)
    if kind == "router":
        return router_case(B=rng.randint(1, 4), T=_log_int(rng, 64, 32768), C=8 * _log_int(rng, 64, 1024),
                           dtype=rng.choice(["bf16", "bf16", "fp32"]))
    if kind == "fp32":
        small = rng.random() < 0.5
        return layer_case("train", T=_log_int(rng, 256, 4096), heads=1 if small else 8,
                          kv=1 if small else rng.choice([2, 8]), D=rng.choice([64, 128]),
                          W=rng.choice([256, 1024]), dtype="fp32", f=round(rng.uniform(0.05, 0.5), 3),
                          separate=rng.random() < 0.3)
    hi = 65536 if kind == "fwd" else 32768
    T = _log_int(rng, 512, hi)
    return layer_case(kind, B=rng.randint(1, 2), T=T, heads=heads, kv=kv, W=rng.choice([1024, 4096]),
                      mask_heads=rng.choice([1, heads]), f=round(rng.uniform(0.05, 0.5), 3),
                      burst=rng.choice([0, 32]), separate=rng.random() < 0.3)


# --------------------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------------------
def _dt(case):
    return torch.bfloat16 if case.get("dtype", "bf16") == "bf16" else torch.float32


def _normals(seed, dtype):
    g = torch.Generator(device=DEV).manual_seed(int(seed) * 1009 + 17)

    def one(*shape):
        return torch.randn(shape, generator=g, device=DEV, dtype=torch.float32).to(dtype)
    return one


def _layer_tensors(case, seed):
    """The tensors of a layer case, in a dict: q, k, v, dO, mask and, with separate modules, qg, kg, vg."""
    one = _normals(seed, _dt(case))
    b, t, hq, hkv, d = case["B"], case["T"], case["heads"], case["kv"], case["D"]
    x = {"q": one(b, t, hq, d), "k": one(b, t, hkv, d), "v": one(b, t, hkv, d)}
    if case["separate"]:
        x.update(qg=one(b, t, hq, d), kg=one(b, t, hkv, d), vg=one(b, t, hkv, d))
    if case["kind"] == "train":
        x["dO"] = one(b, t, hq, d)
    if case["burst"]:
        m = gen.mask_markov(b, case["mask_heads"], t, case["f"], case["burst"], int(seed))
    else:
        m = gen.mask_bernoulli(b, case["mask_heads"], t, case["f"], int(seed))
    x["mask"] = torch.from_numpy(m).to(DEV)
    return x


def _decode_positions(case):
    """Positions of the new tokens: sequences of a batch are of different lengths, from full caches to
    three quarters of the capacity."""
    cap = case["capacity"]
    return [cap - 1 - (i * 977) % max(1, cap // 4) for i in range(case["B"])]


def _decode_routed(case):
    """Which sequences route: `routed` of them, spread over the batch."""
    n, r = case["B"], case["routed"]
    return [(i * r) // n != ((i + 1) * r) // n for i in range(n)]


def _ring_slots(case):
    return (case["W"] + 1 + 31) // 32 * 32


def _decode_tensors(case, seed):
    one = _normals(seed, torch.bfloat16)
    b, cap, hq, hkv = case["B"], case["capacity"], case["heads"], case["kv"]
    x = {"q": one(b, hq, 128), "k": one(b, cap, hkv, 128), "v": one(b, cap, hkv, 128)}
    if case["separate"]:
        x["q_ring"] = one(b, hq, 128)
        x["k_ring"], x["v_ring"] = one(b, _ring_slots(case), hkv, 128), one(b, _ring_slots(case), hkv, 128)
    x["pos"] = torch.tensor(_decode_positions(case), dtype=torch.int32, device=DEV)
    x["mask"] = torch.tensor(_decode_routed(case), dtype=torch.uint8, device=DEV).reshape(b, 1)
    return x


def _router_tensors(case, seed):
    one = _normals(seed, _dt(case))
    x = one(case["B"], case["T"], case["C"])
    w = _normals(seed + 1, torch.float32)(case["C"]) * case["C"] ** -0.5
    return {"x": x, "w": w, "bias": 0.0, "tau": 0.8}     # logits ~ N(0,1): about one token in twelve is routed


def _workspace(nbytes):
    return torch.empty(max(int(nbytes), 16), dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    kind = case["kind"]
    state = {"kind": kind}
    if kind in ("fwd", "train"):
        x = _layer_tensors(case, seed)
        p = B.make_params(case["B"], case["T"], case["heads"], case["kv"], case["D"], case["W"], case["mask_heads"],
                          B.L2A_BF16 if case["dtype"] == "bf16" else B.L2A_FP32)
        state.update(layer=Layer(p, x["q"], x["k"], x["v"], x["mask"], x.get("qg"), x.get("kg"), x.get("vg")),
                     dO=x.get("dO"), separate=case["separate"])
        return state
    if kind == "decode":
        x = _decode_tensors(case, seed)
        hq, hkv, b = case["heads"], case["kv"], case["B"]
        out = lambda: torch.empty(b, hq, 128, dtype=torch.bfloat16, device=DEV)  # noqa: E731
        stat = lambda: torch.empty(b, hq, dtype=torch.float32, device=DEV)  # noqa: E731
        calls = []
        if case["separate"]:
            rp = B.make_params(b, _ring_slots(case), hq, hkv, 128, case["W"], 1,
                               flags=B.L2A_FLAG_SKIP_GLOBAL | B.L2A_FLAG_RING_CACHE)
            calls.append((rp, x["q_ring"], x["k_ring"], x["v_ring"], out(), stat(), None))
            gp = B.make_params(b, case["capacity"], hq, hkv, 128, case["W"], 1, flags=B.L2A_FLAG_SKIP_LOCAL)
            calls.append((gp, x["q"], x["k"], x["v"], out(), None, stat()))
        else:
            p = B.make_params(b, case["capacity"], hq, hkv, 128, case["W"], 1)
            calls.append((p, x["q"], x["k"], x["v"], out(), stat(), stat()))
        state["calls"] = [c + (_workspace(B.lib().l2a_decode_workspace_bytes(ctypes.byref(c[0]))),) for c in calls]
        state.update(pos=x["pos"], mask=x["mask"])
        return state
    x = _router_tensors(case, seed)
    b, t = case["B"], case["T"]
    p = B.make_params(b, t, 1, 1, 128, 0, 1, B.L2A_BF16 if case["dtype"] == "bf16" else B.L2A_FP32)
    state.update(x, p=p, mask=torch.empty(b, 1, t, dtype=torch.uint8, device=DEV),
                 dhat=torch.empty(b, t, device=DEV), logit=torch.empty(b, t, device=DEV))
    return state


def run(state):
    kind = state["kind"]
    if kind == "decode":
        outs = []
        for p, q, k, v, O, lse_l, lse_g, ws in state["calls"]:
            B.l2a_attn_decode(p, q, k, v, state["pos"], state["mask"], O, lse_l, lse_g, workspace=ws)
            outs.append({"O": O, "lse_local": lse_l, "lse_global": lse_g})
        return outs
    if kind == "router":
        B.l2a_router_decide(state["p"], state["x"], state["w"], state["bias"], state["tau"], state["mask"],
                            state["dhat"], state["logit"])
        return {"mask": state["mask"], "dhat": state["dhat"], "logit": state["logit"]}
    lay = state["layer"]
    lay.route()
    lay.forward(save_branches=kind == "train")
    out = {"rows": lay.row_idx, "count": lay.count, "O": lay.O, "lse_local": lay.lse_l, "lse_global": lay.lse_g}
    if kind == "train":
        lay.backward(state["dO"], separate=state["separate"], want_delta=state["separate"])
        out.update(dq=lay.dq, dk=lay.dk, dv=lay.dv)
        if state["separate"]:
            out.update(dqg=lay.dqg, dkg=lay.dkg, dvg=lay.dvg, delta_global=lay.delta_g)
    return out


# --------------------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------------------
def work(case):
    kind = case["kind"]
    if kind == "router":
        n = case["B"] * case["T"]
        e = 2 if case["dtype"] == "bf16" else 4
        return {"bytes": n * (case["C"] * e + 9) + 4 * case["C"], "flops": 2 * n * case["C"]}
    if kind == "decode":
        keys = reads = 0      # with one cache for both branches the window is part of the prefix and read once
        for pos, routed in zip(_decode_positions(case), _decode_routed(case)):
            window, prefix = min(pos, case["W"]) + 1, (pos + 1 if routed else 0)
            keys += window + prefix
            reads += window + prefix if case["separate"] else max(window, prefix)
        heads = case["B"] * case["heads"] * (2 if case["separate"] else 1)
        return {"bytes": reads * case["kv"] * 128 * 2 * 2 + heads * (128 * 2 * 2 + 4),
                "flops": 4 * 128 * case["heads"] * keys}
    b, t, hq, hkv, d = case["B"], case["T"], case["heads"], case["kv"], case["D"]
    w = min(case["W"], t - 1)
    local = b * hq * (t * (w + 1) - w * (w + 1) // 2)
    pairs = local + case["f"] * b * hq * t * (t + 1) / 2
    e = 2 if case["dtype"] == "bf16" else 4
    modules = 2 if case["separate"] else 1
    qs, kvs = b * t * hq * d * e, 2 * b * t * hkv * d * e
    size = b * case["mask_heads"] * t + modules * (qs + kvs) + qs + 2 * 4 * b * hq * t + 4 * case["f"] * b * hq * t
    if kind == "train":
        size += qs + modules * (qs + kvs)      # dO; the gradients of every module's q, k, v
    return {"bytes": size, "flops": (14 if kind == "train" else 4) * d * pairs}


# --------------------------------------------------------------------------------------
# tolerances and the 64-bit answer
# --------------------------------------------------------------------------------------
def tolerance(case):
    """About four times the error that exact() shows for these outputs at this precision.  bf16: outputs are stored
    in 8 bits of mantissa and P, dS enter the products in bf16.  A router's decision may differ where the logit is
    within rounding of the threshold."""
    if case["kind"] == "router":
        return {"rel": 1e-6, "max": 4e-6, "differ": 1e-4}
    if case.get("dtype", "bf16") == "fp32":
        return {"rel": 8e-6, "max": 1e-4}
    if case["kind"] == "train":
        return {"rel": 1.2e-2, "max": 0.6}
    return {"rel": 1e-2, "max": 0.3}


def _branch64(x, suffix, case, local, mask, grads):
    """One branch in 64 bits, plain torch: (out [B,T,H,D], lse [B,H,T], dq, dk, dv, delta [B,H,T])."""
    q, k, v = (x[n + suffix] for n in "qkv")
    b, t, hq, d = q.shape
    hkv, group, scale = k.shape[2], q.shape[2] // k.shape[2], q.shape[3] ** -0.5
    f64 = {"dtype": torch.float64, "device": DEV}
    out = torch.zeros(q.shape, **f64)
    lse = torch.full((b, hq, t), -math.inf, **f64)
    delta = torch.zeros((b, hq, t), **f64)
    dq, dk, dv = (torch.zeros(y.shape, **f64) if grads else None for y in (q, k, v))
    for bi in range(b):
        for h in range(hq):
            hk = h // group
            kk, vv = k[bi, :, hk].double(), v[bi, :, hk].double()
            if local:
                rows = torch.arange(t, device=DEV)
            else:
                rows = mask[bi, 0 if mask.shape[1] == 1 else h].nonzero().reshape(-1)
            at = rows.tolist()
            i = 0
            while i < len(at):
                step = max(64, min(1024, 2 ** 27 // (at[i] + 1)))
                r = rows[i:i + step]
                lo = max(0, at[i] - case["W"]) if local else 0
                hi = at[min(i + step, len(at)) - 1] + 1
                i += step
                qr, kc, vc = q[bi, r, h].double(), kk[lo:hi], vv[lo:hi]
                s = qr @ kc.T
                s *= scale
                j = torch.arange(lo, hi, device=DEV)
                out_of_reach = j[None, :] > r[:, None]
                if local:
                    out_of_reach |= j[None, :] < r[:, None] - case["W"]
                s.masked_fill_(out_of_reach, -math.inf)
                top = s.amax(1, keepdim=True)
                s.sub_(top).exp_()
                total = s.sum(1, keepdim=True)
                s /= total
                lse[bi, h, r] = (top + total.log()).reshape(-1)
                out[bi, r, h] = s @ vc
                if grads:
                    g = x["dO"][bi, r, h].double()
                    dv[bi, lo:hi, hk] += s.T @ g
                    dl = (g * out[bi, r, h]).sum(1, keepdim=True)
                    delta[bi, h, r] = dl.reshape(-1)
                    dp = g @ vc.T
                    dp.sub_(dl).mul_(s).mul_(scale)
                    dq[bi, r, h] = dp @ kc
                    dk[bi, lo:hi, hk] += dp.T @ qr
    return out, lse, dq, dk, dv, delta


def _exact_layer(case, seed):
    x = _layer_tensors(case, seed)
    train, sep = case["kind"] == "train", case["separate"]
    lo = _branch64(x, "", case, True, x["mask"], train)
    gl = _branch64(x, "g" if sep else "", case, False, x["mask"], train)
    out = {"rows": None, "count": None, "O": lo[0] + gl[0], "lse_local": lo[1], "lse_global": gl[1]}
    if train and sep:
        out.update(dq=lo[2], dk=lo[3], dv=lo[4], dqg=gl[2], dkg=gl[3], dvg=gl[4], delta_global=gl[5])
    elif train:
        out.update(dq=lo[2] + gl[2], dk=lo[3] + gl[3], dv=lo[4] + gl[4])
    return out


def _attend64(q, k, v):
    """q [H, D] against k, v [n, Hkv, D] -> (out [H, D], lse [H])"""
    group, outs, lses = q.shape[0] // k.shape[1], [], []
    for h in range(q.shape[0]):
        s = (k[:, h // group].double() @ q[h].double()) * q.shape[1] ** -0.5
        lses.append(torch.logsumexp(s, 0))
        outs.append(torch.softmax(s, 0) @ v[:, h // group].double())
    return torch.stack(outs), torch.stack(lses)


def _exact_decode(case, seed):
    x = _decode_tensors(case, seed)
    b, hq = case["B"], case["heads"]
    f64 = {"dtype": torch.float64, "device": DEV}
    S, A = torch.zeros(b, hq, 128, **f64), torch.zeros(b, hq, 128, **f64)
    ls, la = torch.zeros(b, hq, **f64), torch.full((b, hq), -math.inf, **f64)
    for i, (pos, routed) in enumerate(zip(_decode_positions(case), _decode_routed(case))):
        if case["separate"]:      # slot of token j: j mod slots
            j = torch.arange(max(0, pos - case["W"]), pos + 1, device=DEV) % _ring_slots(case)
            S[i], ls[i] = _attend64(x["q_ring"][i], x["k_ring"][i, j], x["v_ring"][i, j])
        else:
            near = slice(max(0, pos - case["W"]), pos + 1)
            S[i], ls[i] = _attend64(x["q"][i], x["k"][i, near], x["v"][i, near])
        if routed:
            A[i], la[i] = _attend64(x["q"][i], x["k"][i, :pos + 1], x["v"][i, :pos + 1])
    if case["separate"]:
        return [{"O": S, "lse_local": ls, "lse_global": None}, {"O": A, "lse_local": None, "lse_global": la}]
    return [{"O": S + A, "lse_local": ls, "lse_global": la}]


def exact(case, seed):
    if case["kind"] == "decode":
        return _exact_decode(case, seed)
    if case["kind"] == "router":
        x = _router_tensors(case, seed)
        w = x["w"].double()
        logit = torch.stack([torch.cat([part.double() @ w for part in row.split(4096)]) for row in x["x"]]) + x["bias"]
        return {"mask": None, "dhat": torch.sigmoid(logit), "logit": logit}
    return _exact_layer(case, seed)
