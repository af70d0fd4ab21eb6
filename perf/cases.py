"""The calls this library is measured on: what a self-play or analysis host asks of it.

Every case is one network evaluated on one batch of positions through the
public entry points: az_net_load once, then az_eval_batch / az_eval_batch_wdl
on device tensors, or the host submission pipeline on its pinned slot buffers.
The networks are the ones the benchmark and the tests use; batch sizes run
from one position to the 1,024 the headline metric is quoted on.

`exact` is the network's definition in float64 (for int8 and fp8 the quantised
network's: exact sums of code products, float64 requantisation).
"""
import math

import numpy as np
import torch

import paper_2609_37447_amd as az

# Networks: the two residual towers of the benchmark, the small fp32 one, the
# fp8 shape of the tests, and the paper's deployed network.
_PLANES = dict(net="planes", in_planes=20, policy_planes=73, value_relu=0, cap=0.0)
_DEPLOYED = dict(net="deployed", in_planes=52, blocks=14, filters=160, hidden=48, value_relu=1, cap=6.0)


def listed():
    return [
        # The smallest network and call: fp32, 16 positions.  Latency is all.
        dict(_PLANES, name="f32_2x32_b16", dtype="f32", blocks=2, filters=32, hidden=64, batch=16, via="eval"),
        # The float source of a published network on a validation set of 64 positions.
        dict(_PLANES, name="f32_20x128_b64", dtype="f32", blocks=20, filters=128, hidden=128, batch=64, via="eval"),
        # A few games' leaves in bf16.
        dict(_PLANES, name="bf16_20x128_b32", dtype="bf16", blocks=20, filters=128, hidden=128, batch=32, via="eval"),
        # One board per compute unit in bf16.
        dict(_PLANES, name="bf16_20x128_b256", dtype="bf16", blocks=20, filters=128, hidden=128, batch=256, via="eval"),
        # The wide network at the full batch: the largest call.
        dict(_PLANES, name="bf16_24x256_b1024", dtype="bf16", blocks=24, filters=256, hidden=128, batch=1024, via="eval"),
        # The interactive regime: one outstanding batch of 64.
        dict(_PLANES, name="int8_20x128_b64", dtype="int8", blocks=20, filters=128, hidden=128, batch=64, via="eval"),
        # The headline: self-play throughput at the full batch.
        dict(_PLANES, name="int8_20x128_b1024", dtype="int8", blocks=20, filters=128, hidden=128, batch=1024, via="eval"),
        # fp8 on the shallow network it is held to its definition on.
        dict(_PLANES, name="fp8_2x128_b1024", dtype="fp8", blocks=2, filters=128, hidden=64, batch=1024, via="eval",
             in_planes=12, policy_planes=40),
        # The deployed network: interactive, full batch, and bf16 at a ragged batch.
        dict(_DEPLOYED, name="deployed_int8_b64", dtype="int8", batch=64, via="eval"),
        dict(_DEPLOYED, name="deployed_int8_b1024", dtype="int8", batch=1024, via="eval"),
        dict(_DEPLOYED, name="deployed_bf16_b333", dtype="bf16", batch=333, via="eval"),
        # An actor's two outstanding batches of 320, host buffers to host buffers,
        # compact legal-move policy.
        dict(_PLANES, name="pipeline_int8_20x128_2x320", dtype="int8", blocks=20, filters=128, hidden=128, batch=320,
             via="pipeline", slots=2, max_legal=64),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["f32", "bf16", "int8", "int8", "fp8", "deployed", "deployed", "pipeline"])
    most = {"f32": 64 * _macs(listed()[1]), "fp8": 1 << 60}.get(kind, 1024 * _macs(listed()[4]))
    while True:
        if kind == "f32":
            c = dict(_PLANES, dtype="f32", blocks=_log_int(rng, 1, 20), filters=8 * _log_int(rng, 1, 32),
                     hidden=rng.choice([64, 100, 128]), batch=_log_int(rng, 1, 64), via="eval")
        elif kind in ("bf16", "int8"):
            c = dict(_PLANES, dtype=kind, blocks=_log_int(rng, 2, 24), filters=rng.choice([64, 128, 128, 256]),
                     hidden=rng.choice([64, 100, 128, 256]), batch=_log_int(rng, 1, 1024), via="eval",
                     cap=rng.choice([0.0, 6.0]), value_relu=rng.choice([0, 1]))
        elif kind == "fp8":
            c = dict(_PLANES, dtype="fp8", blocks=rng.choice([1, 2]), filters=rng.choice([128, 256]), hidden=64,
                     batch=_log_int(rng, 1, 1024), via="eval", in_planes=rng.choice([12, 20]),
                     policy_planes=rng.choice([40, 73]))
        elif kind == "deployed":
            c = dict(_DEPLOYED, dtype=rng.choice(["int8", "int8", "bf16"]), blocks=rng.randint(2, 14),
                     batch=_log_int(rng, 1, 1024), via="eval")
        else:
            c = dict(_PLANES, dtype="int8", blocks=20, filters=128, hidden=128, batch=_log_int(rng, 16, 1024),
                     via="pipeline", slots=rng.choice([1, 2, 4]), max_legal=rng.choice([64, 256]))
        if _macs(c) * c["batch"] * c.get("slots", 1) <= most:
            return c


# --------------------------------------------------------------------------- #
# Sizes
# --------------------------------------------------------------------------- #
_D, _V = 128, 2           # the deployed network's token width and value channels


def _moves(c):
    return 1880 if c["net"] == "deployed" else c["policy_planes"] * 64


def _pools(c, j):
    return c["net"] == "deployed" and j % 2 == 1


def _layers(c):
    """(name, shape) in the weight blob's order."""
    C, F, H = c["in_planes"], c["filters"], c["hidden"]
    out = [("stem.w", (F, C, 3, 3)), ("stem.b", (F,))]
    for j in range(c["blocks"]):
        out += [(f"{j}.w1", (F, F, 3, 3)), (f"{j}.b1", (F,))]
        if _pools(c, j):
            out += [(f"{j}.pool", (F - F // 4, F // 4 * 2))]
        out += [(f"{j}.w2", (F, F - F // 4 if _pools(c, j) else F, 3, 3)), (f"{j}.b2", (F,))]
    if c["net"] == "deployed":
        out += [("embed.w", (_D, F)), ("embed.b", (_D,)), ("query.w", (_D, _D)), ("query.b", (_D,)),
                ("key.w", (_D, _D)), ("key.b", (_D,)), ("promo.w", (4, _D)),
                ("value.w", (_V, F)), ("value.b", (_V,)), ("fc1.w", (H, _V * 64)), ("fc1.b", (H,)),
                ("fc2.w", (3, H)), ("fc2.b", (3,))]
    else:
        P = c["policy_planes"]
        out += [("policy.w", (P, F)), ("policy.b", (P,)), ("value.w", (1, F)), ("value.b", (1,)),
                ("fc1.w", (H, 64)), ("fc1.b", (H,)), ("fc2.w", (1, H)), ("fc2.b", (1,))]
    return out


def _macs(c):
    """Multiply-accumulates of one position (no padding, no halo)."""
    n = 0
    for name, s in _layers(c):
        if len(s) == 4:
            n += 64 * s[0] * s[1] * 9
        elif len(s) == 2:
            per_square = name.split(".")[0] in ("policy", "value", "embed", "query", "key")
            n += s[0] * s[1] * (64 if per_square else 8 if name == "promo.w" else 1)
    return n + (64 * 64 * _D if c["net"] == "deployed" else 0)


def work(case):
    n = case["batch"] * case.get("slots", 1)
    policy = case["max_legal"] + 1 if case["via"] == "pipeline" else _moves(case)
    wdl = 3 if case["net"] == "deployed" else 0
    es = {"f32": 4, "bf16": 2, "int8": 1, "fp8": 1}[case["dtype"]]
    weights = sum(int(np.prod(s)) * (es if len(s) == 4 else 4) for _, s in _layers(case))
    return {"bytes": n * (case["in_planes"] * 256 + _moves(case) + 4 * (policy + 1 + wdl)) + weights,
            "flops": 2 * n * _macs(case)}


def tolerance(case):
    # From the distance to `exact`, times four.  fp32: 1e-6.  bf16: 2e-3 to 5e-3.
    # fp8: 6e-3 (policy) and 1.6e-2 (value): its matrix instruction truncates.
    # int8: 1e-7 to 1e-5; but its bf16 stem is summed in fp32, and another order of
    # those sums can move one stem code across a rounding boundary, which shifts
    # that one position by up to 0.005 (2e-3 of a batch).
    return {"f32": {"rel": 1e-5, "max": 1e-3}, "int8": {"rel": 2e-3, "max": 0.5},
            "bf16": {"rel": 2e-2, "max": 0.9}, "fp8": {"rel": 3e-2, "max": 0.9}}[case["dtype"]]


# --------------------------------------------------------------------------- #
# Inputs
# --------------------------------------------------------------------------- #
def _gen(case, seed, what):
    return torch.Generator(device="cuda").manual_seed(1000003 * seed + what)


def _weights(case, seed):
    """{name: float32 array}: N(0, 2 / fan_in), biases N(0, 0.1^2), the residual
    branch's scale folded in, heads scaled so that policies and values are
    spread as a trained network's are; on the bf16 grid except for fp32."""
    g = _gen(case, seed, 1)
    W = {}
    for name, s in _layers(case):
        x = torch.randn(s, generator=g, device="cuda")
        fan = s[1] * 9 if len(s) == 4 else s[-1]
        x = x * (0.1 if len(s) == 1 else math.sqrt(2.0 / fan))
        if name.endswith((".w2", ".b2")):
            x = x / math.sqrt(case["blocks"])
        if name.startswith("embed"):
            x = x / 4
        if name.startswith("fc2"):
            x = x / 8
        W[name] = x if case["dtype"] == "f32" else x.bfloat16().float()
    return W


def _pieces(g, n):
    """One-hot pieces [n, 12, 64]: 16 to 32 on distinct squares."""
    rank = torch.rand((n, 64), generator=g, device="cuda").argsort(1).argsort(1)
    there = rank < torch.randint(16, 33, (n, 1), generator=g, device="cuda")
    kind = torch.randint(0, 12, (n, 64), generator=g, device="cuda")
    return torch.nn.functional.one_hot(kind, 12).transpose(1, 2) * there[:, None]


def _planes(case, g, n):
    """Side-to-move planes: pieces, then constant flags; the deployed network's
    52 add occupancy, recent moves' squares, the checkerboard and whole-number
    counts."""
    C = case["in_planes"]
    x = torch.zeros((n, C, 64), device="cuda")
    x[:, :12] = _pieces(g, n).float()
    flags = torch.randint(0, 2, (n, C, 1), generator=g, device="cuda").float()
    if case["net"] != "deployed":
        x[:, 12:] = flags[:, 12:].expand(-1, -1, 64)
        return x.reshape(n, C, 8, 8)
    x[:, 12:16] = flags[:, 12:16]
    x[:, 16], x[:, 17] = x[:, 0:6].amax(1), x[:, 6:12].amax(1)
    x[:, 20:22] = flags[:, 20:22]
    square = torch.randint(0, 64, (n, 18), generator=g, device="cuda")
    marks = torch.nn.functional.one_hot(square, 64).float()
    moves = torch.randint(0, 9, (n, 1), generator=g, device="cuda")
    x[:, 22:38] = marks[:, :16] * (torch.arange(16, device="cuda") // 2 < moves)[:, :, None]
    x[:, 18] = marks[:, 16] * x[:, 17]
    x[:, 19] = marks[:, 17] * flags[:, 19]
    sq = torch.arange(64, device="cuda")
    x[:, 38] = ((sq // 8 + sq % 8) % 2 == 0).float()
    x[:, 39] = flags[:, 39]
    own, their = x[:, 0:6].sum(2), x[:, 6:12].sum(2)
    x[:, 40:46] = (own - their)[:, :, None]
    x[:, 46] = torch.randint(0, 101, (n, 1), generator=g, device="cuda").float()
    x[:, 47:52] = own[:, :5, None]
    return x.reshape(n, C, 8, 8)


def _legal(case, g, n):
    """20 to 40 distinct legal moves a position."""
    M = _moves(case)
    at = torch.rand((n, M), generator=g, device="cuda").topk(40, dim=1).indices
    keep = torch.arange(40, device="cuda") < torch.randint(20, 41, (n, 1), generator=g, device="cuda")
    return torch.zeros((n, M), dtype=torch.uint8, device="cuda").scatter_(1, at, keep.to(torch.uint8))


def _inputs(case, seed):
    n = case["batch"] * case.get("slots", 1)
    g = _gen(case, seed, 2)
    return _planes(case, g, n), _legal(case, g, n)


def _scales(case, W, seed):
    """(per-channel weight scales, activation scales): largest magnitudes, the
    activations' over 32 calibration positions, or the cap where there is one."""
    if case["dtype"] not in ("int8", "fp8"):
        return None, None
    qmax = 127.0 if case["dtype"] == "int8" else 448.0
    ws = torch.stack([W[f"{j}.w{i}"].abs().flatten(1).amax(1) for j in range(case["blocks"]) for i in (1, 2)])
    ws = torch.where(ws > 0, ws / qmax, torch.ones_like(ws))
    k = 2 * case["blocks"] + 1
    if case["cap"]:
        a = torch.full((k,), case["cap"] / qmax)
    else:
        peaks = []
        _tower(dict(case, dtype="float"), W, _planes(case, _gen(case, seed, 3), 32), None, None, peaks)
        m, e = np.frexp(np.array(peaks) / qmax)
        # Rounded up, so that no last bits of a sum are in it, and off the grid that
        # bf16 weights and biases put the stem's sums on: no quotient is a tie.
        a = torch.tensor(np.ldexp(np.ceil(m * 256) / 256, e) * (1 + math.pi / 1000))
    return ws.float().cpu().numpy(), a.float().numpy()


class _Held(np.ndarray):
    """A view of a slot's pinned buffer that keeps the pipeline it belongs to."""
    owner = None


class _State:
    def __init__(self, net):
        self.net, self.pipe = net, None

    def __del__(self):
        if self.pipe is not None:
            self.pipe.close()
        if self.net is not None:
            torch.cuda.synchronize()
            az.az_net_free(self.net)


def prepare(case, seed):
    W = _weights(case, seed)
    ws, acs = _scales(case, W, seed)
    deployed = case["net"] == "deployed"
    n = case["batch"]
    spec = az.make_spec(case["in_planes"], case["blocks"], case["filters"],
                        0 if deployed else case["policy_planes"], case["hidden"],
                        value_conv_relu=case["value_relu"], act_cap=case["cap"], max_batch=n,
                        pool_every=2 if deployed else 0,
                        policy_head=az.AZ_POLICY_FROMTO if deployed else az.AZ_POLICY_PLANES,
                        token_dim=_D if deployed else 0,
                        value_head=az.AZ_VALUE_WDL if deployed else az.AZ_VALUE_TANH,
                        value_channels=_V if deployed else 1)
    blob = torch.cat([W[name].flatten() for name, _ in _layers(case)]).cpu().numpy()
    s = _State(az.az_net_load(spec, blob, case["dtype"], ws, acs))
    planes, legal = _inputs(case, seed)
    if case["via"] == "pipeline":
        s.pipe = az.Pipeline(s.net, spec, n, case["slots"], max_legal=case["max_legal"])
        for k, (p, l, _, _, _) in enumerate(s.pipe.views):
            p[:] = planes[k * n:(k + 1) * n].cpu().numpy()
            l[:] = legal[k * n:(k + 1) * n].cpu().numpy()
        s.batch = n
        s.outputs = []
        for _, _, po, va, co in s.pipe.views:
            s.outputs.append({"policy": po.view(_Held), "value": va.view(_Held), "count": co.view(_Held)})
        return s
    s.planes, s.legal = planes, legal
    s.policy = torch.empty((n, _moves(case)), device="cuda")
    s.value = torch.empty((n,), device="cuda")
    s.wdl = torch.empty((n, 3), device="cuda") if deployed else None
    return s


def _hold(a, owner):
    v = a.view()
    v.owner = owner
    return v


def run(s):
    if s.pipe is not None:
        for k in range(len(s.pipe.views)):
            s.pipe.submit(k, s.batch)
        for k in range(len(s.pipe.views)):
            s.pipe.wait(k)
        return [{k: _hold(v, s) for k, v in out.items()} for out in s.outputs]
    az.eval_tensors(s.net, s.planes, s.legal, s.policy, s.value, wdl=s.wdl)
    out = {"policy": s.policy, "value": s.value}
    return out if s.wdl is None else dict(out, wdl=s.wdl)


# --------------------------------------------------------------------------- #
# The definition in float64
# --------------------------------------------------------------------------- #
def _conv(x, w):
    """3x3, zero pad: x [n, C, 64] float64, w [F, C, 3, 3]."""
    n, C, _ = x.shape
    cols = torch.nn.functional.unfold(x.reshape(n, C, 8, 8), 3, padding=1)       # [n, 9 C, 64]
    y = w.reshape(w.shape[0], -1).double() @ cols.transpose(0, 1).reshape(9 * C, n * 64)
    return y.reshape(w.shape[0], n, 64).transpose(0, 1)


def _mix(w, x):
    """1x1: w [F, C], x [n, C, 64]."""
    n, C, S = x.shape
    return (w.double() @ x.transpose(0, 1).reshape(C, n * S)).reshape(w.shape[0], n, S).transpose(0, 1)


def _round_e4m3(x):
    _, e = torch.frexp(x)
    step = torch.ldexp(torch.ones_like(x), torch.clamp(e - 1, min=-6) - 3)
    return torch.round(x / step) * step


def _tower(case, W, planes, ws, acs, peaks=None):
    """The final tensor h [n, F, 64] in float64; peaks collects every tensor's
    largest value."""
    quant = ws is not None
    qmax = 127.0 if case["dtype"] == "int8" else 448.0
    grid = torch.round if case["dtype"] == "int8" else _round_e4m3

    def act(y):
        y = y.clamp(min=0)
        return y.clamp(max=case["cap"]) if case["cap"] else y

    def out(y, k):          # a stored tensor's values
        y = act(y)
        if quant:
            a = float(acs[k])
            y = grid(y / a).clamp(max=qmax) * a
        if peaks is not None:
            peaks.append(float(y.max()))
        return y

    def conv(x, n, name):
        w = W[name].double()
        if not quant:
            return _conv(x, w)
        a, s = float(acs[n]), torch.tensor(ws[n], device="cuda").double()
        q = grid(w / s[:, None, None, None]).clamp(-qmax, qmax)
        # codes (rounded back off a) times codes: exact in float64
        return _conv(grid(x / a), q) * (a * s)[:, None]

    h = out(_conv(planes.reshape(len(planes), -1, 64).double(), W["stem.w"]) + W["stem.b"].double()[:, None], 0)
    for j in range(case["blocks"]):
        z = conv(h, 2 * j, f"{j}.w1") + W[f"{j}.b1"].double()[:, None]
        if _pools(case, j):
            f = z.shape[1] - z.shape[1] // 4
            pc = act(z[:, f:])
            z = z[:, :f] + torch.cat([pc.mean(2), pc.amax(2)], 1) .matmul(W[f"{j}.pool"].double().T)[:, :, None]
        t = out(z, 2 * j + 1)
        h = out(h + conv(t, 2 * j + 1, f"{j}.w2") + W[f"{j}.b2"].double()[:, None], 2 * j + 2)
    return h


def _actions():
    at = []
    for f in range(64):
        for t in range(64):
            dr, dc = abs(f // 8 - t // 8), abs(f % 8 - t % 8)
            if f != t and (dr == 0 or dc == 0 or dr == dc or {dr, dc} == {1, 2}):
                at.append((f * 64 + t, -1))
    for f in range(48, 56):
        for t in range(56, 64):
            if abs(f % 8 - t % 8) <= 1:
                at += [(f * 64 + t, (t - 56) * 4 + k) for k in range(4)]
    return at


def _soft(z, legal):
    z = torch.where(legal != 0, z, torch.full_like(z, -math.inf))
    p = torch.exp(z - z.amax(1, keepdim=True))
    return p / p.sum(1, keepdim=True)


def _whole(case, W, planes, legal, ws, acs):
    b = lambda name: W[name].double()  # noqa: E731
    h = _tower(case, W, planes, ws, acs)
    n = len(planes)
    u = _mix(b("value.w"), h) + b("value.b")[:, None]
    u = (u.clamp(min=0) if case["value_relu"] else u).reshape(n, -1)
    y = (u @ b("fc1.w").T + b("fc1.b")).clamp(min=0) @ b("fc2.w").T + b("fc2.b")
    if case["net"] != "deployed":
        z = (_mix(b("policy.w"), h) + b("policy.b")[:, None]).reshape(n, -1)
        return {"policy": _soft(z, legal), "value": torch.tanh(y[:, 0])}
    tok = (_mix(b("embed.w"), h) + b("embed.b")[:, None]).clamp(min=0)
    q, k = (_mix(b(m + ".w"), tok) + b(m + ".b")[:, None] for m in ("query", "key"))
    s = q.transpose(1, 2).contiguous().matmul(k.contiguous()) / math.sqrt(_D)
    o = _mix(b("promo.w"), k[:, :, 56:].contiguous())                            # [n, 4, 8]
    at = torch.tensor(_actions(), device="cuda")
    z = s.reshape(n, -1)[:, at[:, 0]]
    off = o.transpose(1, 2).reshape(n, 32)[:, at[:, 1].clamp(min=0)]
    wdl = torch.softmax(y, 1)
    return {"policy": _soft(z + torch.where(at[:, 1] >= 0, off, torch.zeros_like(off)), legal),
            "value": wdl[:, 0] - wdl[:, 2], "wdl": wdl}


def exact(case, seed):
    W = _weights(case, seed)
    ws, acs = _scales(case, W, seed)
    planes, legal = _inputs(case, seed)
    parts = [_whole(case, W, planes[i:i + 128], legal[i:i + 128], ws, acs) for i in range(0, len(planes), 128)]
    full = {k: torch.cat([p[k] for p in parts]) for k in parts[0]}
    if case["via"] != "pipeline":
        return full
    n, m = case["batch"], case["max_legal"]
    out = []
    for k in range(case["slots"]):
        p, l = full["policy"][k * n:(k + 1) * n].cpu().numpy(), legal[k * n:(k + 1) * n].cpu().numpy()
        rows = np.zeros((n, m))
        for i in range(n):
            v = p[i][l[i] != 0]
            rows[i, :len(v)] = v
        out.append({"policy": rows, "value": full["value"][k * n:(k + 1) * n].cpu().numpy(),
                    "count": (l != 0).sum(1).astype(np.int32)})
    return out
