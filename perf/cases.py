"""Performance cases of the lossy data-parallel step.

What a program of this framework does on the GPU, through its public entry
points: the fused step at the sizes of the repository's workloads (the
smallest, where launches count, up to a 64-worker ZeRO-2 shard), the same with
network-sized packets, with the delivery variants and with Algorithm 1's stale
fill, and the one-stage calls a program makes when it moves the packets itself
between the gradient half and the broadcast half.

A case is a dict of plain values; see `listed` for what each stands for and
`draw` for the ranges.  Every size is in elements unless its name says bytes.
"""
import math

import numpy as np
import torch

import paper_2507_07114_amd as ll

SGD = dict(opt="sgd", lr=0.01)
MOMENTUM = dict(opt="momentum", lr=0.01, momentum=0.9)
ADAM = dict(opt="adam", lr=3e-4, beta1=0.9, beta2=0.95, eps=1e-8)
BURSTS = dict(loss="gilbert_elliott", p_gb=0.01, p_bg=0.2, loss_good=0.0, loss_bad=0.5)

# Step index of a state's first pass: a program in the middle of its run.
FIRST_STEP = 9


def _bernoulli(p):
    return dict(loss="bernoulli", p=p)


def _step(name, n, d, packet, dtype, loss, opt, **more):
    """One lossy_step_fused call.  ld_to: rows are padded to a multiple of
    this many elements; masks_out: the caller keeps the routing log (masks
    and counts); drift: the call also measures the replicas' drift."""
    c = dict(name=name, kind="step", n=n, d=d, packet=packet, gdtype=dtype, rdtype=dtype,
             ld_to=256, estimator="arrived_mean", owner=-1, reliable_every=0, parity=0,
             ages=False, drift=True, masks_out=True)
    c.update(loss)
    c.update(opt)
    c.update(more)
    return c


def _stage(name, kind, n, d, packet, dtype, loss, opt=None):
    c = dict(name=name, kind=kind, n=n, d=d, packet=packet, gdtype=dtype, rdtype=dtype, ld_to=256)
    c.update(loss)
    c.update(opt or {})
    return c


def listed():
    return [
        # The smallest step a program makes (4 workers, 1 Mi fp32, a few tens
        # of MB): launches and the host's share of a call.
        _step("step_n4_d1m_f32_sgd", 4, 1_048_576, 1024, "f32", _bernoulli(0.1), SGD),
        # One node's worth of workers, mixed precision, Adam: an ordinary step.
        _step("step_n8_d16m_bf16_adam", 8, 16_777_216, 2048, "bf16", _bernoulli(0.01), ADAM),
        # The paper's set-up: 64 workers, one ZeRO-2 shard of a 6.74e9-element
        # model; the benchmark's step and the largest case.
        _step("step_n64_d105m_bf16_adam", 64, 105_250_000, 4096, "bf16", _bernoulli(0.1), ADAM),
        # A quarter Gi of fp32 elements per worker under bursty loss.
        _step("step_n16_d256m_f32_ge", 16, 268_435_456, 4096, "f32", BURSTS, MOMENTUM),
        # Long drift study: 64 fp32 replicas, drift after every step.
        _step("step_n64_d48m_f32_sgd", 64, 50_331_648, 2048, "f32", _bernoulli(0.1),
              dict(SGD, lr=1e-3)),
        # Packets as an Ethernet link cuts them, 1500 bytes = 750 bf16
        # elements (not a multiple of 8), and an odd shard length.
        _step("step_n16_d16m_mtu1500_bf16", 16, 16_777_259, 750, "bf16", _bernoulli(0.02), ADAM),
        # Every delivery option at once: parity packets, an owner row, some
        # packets on a reliable channel, Horvitz-Thompson weights, ages; an
        # eighth of the 64-worker shard.
        _step("step_n64_d13m_delivery_bf16", 64, 13_156_250, 4096, "bf16", _bernoulli(0.1), ADAM,
              estimator="horvitz_thompson", owner=0, reliable_every=10, parity=8, ages=True),
        # Algorithm 1 (lost contributions replaced by the last that arrived),
        # without drift or a routing log.
        _step("step_n32_d8m_stale_fill_bf16", 32, 8_388_608, 2048, "bf16", _bernoulli(0.1),
              MOMENTUM, estimator="stale_fill", drift=False, masks_out=False),
        # The gradient half by itself: masks and aggregate, a quarter of the shard.
        _stage("aggregate_n64_d26m_bf16", "aggregate", 64, 26_312_500, 4096, "bf16",
               _bernoulli(0.1)),
        # The owner's update of the whole shard by itself.
        _stage("update_d105m_adam", "update", 1, 105_250_000, 4096, "f32", _bernoulli(0.1), ADAM),
        # The broadcast half by itself.
        _stage("broadcast_n64_d26m_bf16", "broadcast", 64, 26_312_500, 4096, "bf16",
               _bernoulli(0.1)),
        # Drift of replicas that a program holds, measured between steps.
        _stage("drift_n64_d26m_bf16", "drift", 64, 26_312_500, 4096, "bf16", _bernoulli(0.1)),
    ]


# Row bytes (both directions) of the largest drawn case: under half of the
# largest listed one's.
_MOST_BYTES = 12e9


def draw(rng):
    """A case of the listed ones' ranges: 2 to 96 workers, shards of 32 Ki to
    105 M elements, packets of 256 to 8192 elements and Ethernet sizes."""
    kind = rng.choice(["step"] * 7 + ["aggregate", "update", "broadcast", "drift"])
    n = int(round(math.exp(rng.uniform(math.log(2), math.log(96)))))
    gdtype = rng.choice(["bf16", "bf16", "f32"])
    rdtype = gdtype if rng.random() < 0.85 else rng.choice(["bf16", "f32"])
    per_elem = n * ((2 if gdtype == "bf16" else 4) + (2 if rdtype == "bf16" else 4))
    top = min(105_250_000, _MOST_BYTES / (per_elem if kind != "update" else 1))
    d = int(math.exp(rng.uniform(math.log(32_768), math.log(top))))
    if rng.random() < 0.5:  # a shard cut at a round size, else any length
        d -= d % 1024
    what = rng.random()
    if what < 0.6:
        packet = rng.choice([256, 512, 1024, 2048, 4096, 8192])
    elif what < 0.75:  # 1500- and 9000-byte Ethernet payloads
        packet = rng.choice([375, 750, 2250, 4500])
    else:
        packet = rng.randrange(256, 8192)
    opt = dict(rng.choice([SGD, MOMENTUM, ADAM]))
    ge = rng.random() < 0.25
    loss = dict(BURSTS) if ge else _bernoulli(rng.choice([0.0, 0.01, 0.05, 0.1, 0.2]))
    if kind != "step":
        c = _stage("", kind, 1 if kind == "update" else n, d, packet, gdtype, loss,
                   opt if kind == "update" else None)
        c["rdtype"] = rdtype
    else:
        est = rng.choice(["arrived_mean"] * 4 + ["horvitz_thompson", "stale_fill"])
        c = _step("", n, d, packet, gdtype, loss, opt, rdtype=rdtype, estimator=est,
                  owner=rng.choice([-1, -1, 0]), reliable_every=rng.choice([0, 0, 10]),
                  parity=0 if ge else rng.choice([0, 0, 0, 4, 8]), ages=rng.random() < 0.25,
                  drift=rng.random() < 0.6, masks_out=rng.random() < 0.5)
    c["ld_to"] = rng.choice([256, 8])
    del c["name"]
    return c


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
_DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16}


def _packets(c):
    return (c["d"] + c["packet"] - 1) // c["packet"]


def _loss_spec(c, seed):
    if c["loss"] == "bernoulli":
        return ll.bernoulli(c["p"], seed=seed)
    return ll.gilbert_elliott(c["p_gb"], c["p_bg"], c["loss_good"], c["loss_bad"], seed=seed)


def _opt_spec(c):
    if c["opt"] == "sgd":
        return ll.sgd(c["lr"])
    if c["opt"] == "momentum":
        return ll.sgd_momentum(c["lr"], c["momentum"])
    return ll.adam(c["lr"], c["beta1"], c["beta2"], c["eps"])


def _normal(gen, d, std):
    return torch.randn(d, generator=gen, device="cuda", dtype=torch.float32).mul_(std)


def _rows(gen, c, dtype, fill):
    """[n][ld] rows of `dtype`, row i from fill(i); padding is zero."""
    ld = -(-c["d"] // c["ld_to"]) * c["ld_to"]
    out = torch.zeros((c["n"], ld), dtype=_DTYPE[dtype], device="cuda")
    for i in range(c["n"]):
        out[i, : c["d"]].copy_(fill(i))
    return out


def prepare(case, seed):
    c, n, d, P = case, case["n"], case["d"], _packets(case)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed * 7919 + 11)
    s = dict(case=c, step=FIRST_STEP, seed=seed)
    s["loss"] = _loss_spec(c, seed)
    theta = s["theta"] = _normal(gen, d, 0.02)
    grads = lambda: _rows(gen, c, c["gdtype"], lambda i: _normal(gen, d, 1e-3))  # noqa: E731
    u8 = lambda *shape: torch.zeros(shape, dtype=torch.uint8, device="cuda")  # noqa: E731
    if c["kind"] in ("step", "update"):
        s["opt"] = _opt_spec(c)
        s["m"] = _normal(gen, d, 3e-4) if c["opt"] != "sgd" else None
        s["v"] = _normal(gen, d, 1e-3).square_() if c["opt"] == "adam" else None
    if c["kind"] in ("step", "aggregate"):
        s["grads"] = grads()
    if c["kind"] in ("step", "broadcast", "drift"):
        # replicas a little behind the master, each by its own amount
        s["replicas"] = _rows(gen, c, c["rdtype"], lambda i: _normal(gen, d, 3e-4).add_(theta))
    if c["kind"] in ("aggregate", "update"):
        s["g_hat"] = _normal(gen, d, 1e-3)
    if c["kind"] in ("aggregate", "broadcast", "drift"):
        s["arrived"] = u8(n, P)
        s["ge_state"] = u8(n)
        s["mask_ws"] = u8(max(ll.ll_masks_workspace_bytes(n, P), 256))
        s["counts"] = torch.zeros(P, dtype=torch.int32, device="cuda")
    if c["kind"] == "drift":  # the masks of the broadcast that came before
        ll.ll_masks(n, P, s["step"], ll.LL_DIR_BCAST, s["loss"], s["arrived"],
                    ge_state=s["ge_state"], workspace=s["mask_ws"])
    if c["kind"] in ("step", "drift"):
        s["drift"] = ll.drift_buffer()
        s["workspace"] = u8(max(ll.ll_workspace_bytes(n, d, c["packet"]), 256))
    if c["kind"] == "step":
        s["ge_g"], s["ge_b"] = u8(n), u8(n)
        s["arrived_g"] = u8(n, P) if c["masks_out"] else None
        s["arrived_b"] = u8(n, P) if c["masks_out"] else None
        s["counts"] = torch.zeros(P, dtype=torch.int32, device="cuda") if c["masks_out"] else None
        s["reliable"] = None
        if c["reliable_every"]:
            s["reliable"] = u8(P)
            s["reliable"][:: c["reliable_every"]] = 1
        s["g_prev"] = grads() if c["estimator"] == "stale_fill" else None
        s["ages"] = torch.zeros((n, P), dtype=torch.int16, device="cuda") if c["ages"] else None
        s["ext"] = ll.ext(c["estimator"], owner=c["owner"], reliable=s["reliable"],
                          g_prev=s["g_prev"], ages=s["ages"], parity_group=c["parity"])
    return s


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def _drift_out(buf):
    return dict(drift=buf[:4], drift_counts=buf.view(torch.int64)[4:])


def run(s):
    c = s["case"]
    n, d, L, P, step = c["n"], c["d"], c["packet"], _packets(c), s["step"]
    if c["kind"] == "step":
        ll.lossy_step_fused(
            d=d, packet=L, step=step, loss_g=s["loss"], loss_b=s["loss"], grads=s["grads"],
            opt=s["opt"], theta=s["theta"], replicas=s["replicas"], m=s["m"], v=s["v"],
            ge_state_g=s["ge_g"], ge_state_b=s["ge_b"], arrived_g=s["arrived_g"],
            arrived_b=s["arrived_b"], counts=s["counts"], workspace=s["workspace"],
            drift=s["drift"] if c["drift"] else None, ext=s["ext"])
        s["step"] = step + 1
        out = {k: s[k] for k in ("theta", "m", "v", "replicas", "arrived_g", "arrived_b",
                                 "counts", "ge_g", "ge_b", "g_prev", "ages")}
        if c["drift"]:
            out.update(_drift_out(s["drift"]))
        return out
    if c["kind"] == "aggregate":
        ll.ll_masks(n, P, step, ll.LL_DIR_GRAD, s["loss"], s["arrived"], ge_state=s["ge_state"],
                    workspace=s["mask_ws"])
        ll.lossy_aggregate(s["grads"], s["arrived"], d=d, packet=L, g_hat=s["g_hat"],
                           counts=s["counts"])
        s["step"] = step + 1
        return {k: s[k] for k in ("arrived", "ge_state", "g_hat", "counts")}
    if c["kind"] == "update":
        ll.shard_step(s["opt"], step, s["theta"], s["g_hat"], m=s["m"], v=s["v"], d=d)
        s["step"] = step + 1
        return {k: s[k] for k in ("theta", "m", "v")}
    if c["kind"] == "broadcast":
        ll.ll_masks(n, P, step, ll.LL_DIR_BCAST, s["loss"], s["arrived"], ge_state=s["ge_state"],
                    workspace=s["mask_ws"])
        ll.lossy_broadcast(s["theta"], s["replicas"], s["arrived"], d=d, packet=L)
        s["step"] = step + 1
        return {k: s[k] for k in ("arrived", "ge_state", "replicas")}
    ll.drift_stats(s["replicas"], d=d, packet=L, workspace=s["workspace"], out=s["drift"],
                   theta=s["theta"], arrived_bc=s["arrived"])
    return _drift_out(s["drift"])


# ---------------------------------------------------------------------------
# What one pass cannot do without
# ---------------------------------------------------------------------------
def _arrival(c):
    if c["loss"] == "bernoulli":
        q = 1.0 - c["p"]
    else:
        bad = c["p_gb"] / (c["p_gb"] + c["p_bg"])
        q = 1.0 - (bad * c["loss_bad"] + (1.0 - bad) * c["loss_good"])
    if c.get("parity"):
        q += (1.0 - q) * q ** c["parity"]
    if c.get("reliable_every"):
        q += (1.0 - q) / c["reliable_every"]
    if c.get("owner", -1) >= 0:
        q += (1.0 - q) / c["n"]
    return q


def work(case):
    c, n, d, P, q = case, case["n"], case["d"], _packets(case), _arrival(case)
    eg, er = (2 if c[k] == "bf16" else 4 for k in ("gdtype", "rdtype"))
    vectors = {"sgd": 1, "momentum": 2, "adam": 3}.get(c.get("opt"), 0)
    update = 2 * 4 * vectors * d
    update_flops = {0: 0, 1: 2, 2: 4, 3: 14}[vectors] * d
    if c["kind"] == "update":
        return dict(bytes=update + 4 * d, flops=update_flops)
    if c["kind"] == "aggregate":
        return dict(bytes=n * d * q * eg + 4 * d + n * P + 4 * P, flops=n * d * q + d)
    if c["kind"] == "broadcast":
        return dict(bytes=n * d * q * er + 4 * d + n * P, flops=d)
    if c["kind"] == "drift":
        return dict(bytes=n * d * er + 4 * d + n * P, flops=6 * n * d)
    rows = n * d * q * eg + n * d * q * er
    flops = n * d * q + d + update_flops
    if c["estimator"] == "stale_fill":  # lost rows from g_prev, arrived ones into it
        rows += n * d * eg
        flops += n * d * (1 - q)
    if c["drift"]:
        rows += n * d * (1 - q) * er
        flops += 6 * n * d * (1 - q)
    masks = 2 * n * P if c["masks_out"] else 0
    return dict(bytes=rows + update + masks + (4 * n * P if c["ages"] else 0), flops=flops)


def tolerance(case):
    # fp32 sums of up to 96 terms in another order move theta, the moments and
    # the drift figures by 1e-7 to 1e-6 of their size; where a bf16 replica
    # value then rounds the other way it moves by 2^-8 of itself.
    if "bf16" in (case["rdtype"] if case["kind"] in ("step", "broadcast", "drift") else "f32",):
        return {"rel": 1e-4, "max": 1e-2}
    return {"rel": 1e-5}


# ---------------------------------------------------------------------------
# The same in 64 bits, with plain torch
# ---------------------------------------------------------------------------
_LOW = 0xFFFFFFFF


def _signed(x):
    return x - (1 << 64) if x >= 1 << 63 else x


def _mul_high(a, x):
    """High 64 bits of the unsigned product of constant a and tensor x (64-bit
    patterns in int64)."""
    al, ah = a & _LOW, a >> 32
    xl, xh = x & _LOW, (x >> 32) & _LOW
    mid = xh * al + (((xl * al) >> 32) & _LOW)
    low = xl * ah + (mid & _LOW)
    return xh * ah + ((mid >> 32) & _LOW) + ((low >> 32) & _LOW)


def _words(n, P, step, direction, seed):
    """Top halves of words 0 and 1 of Philox4x64-10 at (k, i, step, direction), [n][P]."""
    m0, m1 = 0xD2E7470EE14C6C93, 0xCA5A826395121157
    c0 = torch.arange(P, device="cuda").expand(n, P).contiguous()
    c1 = torch.arange(n, device="cuda")[:, None].expand(n, P).contiguous()
    c2 = torch.full_like(c0, step)
    c3 = torch.full_like(c0, direction)
    k0, k1 = seed, 0
    for _ in range(10):
        h0, l0 = _mul_high(m0, c0), c0 * _signed(m0)
        h1, l1 = _mul_high(m1, c2), c2 * _signed(m1)
        c0, c1, c2, c3 = h1 ^ c1 ^ _signed(k0), l1, h0 ^ c3 ^ _signed(k1), l0
        k0 = (k0 + 0x9E3779B97F4A7C15) & ((1 << 64) - 1)
        k1 = (k1 + 0xBB67AE8584CAA73B) & ((1 << 64) - 1)
    return (c0 >> 32) & _LOW, (c1 >> 32) & _LOW


def _threshold(p):
    return math.ceil(p * 4294967296.0)


def _masks(c, step, direction, seed, reliable):
    """(arrived bool [n][P], end state uint8 [n]) of one direction."""
    n, P = c["n"], _packets(c)
    w0, w1 = _words(n, P, step, direction, seed)
    state = torch.zeros(n, dtype=torch.uint8)
    sure = torch.zeros((n, P), dtype=torch.bool, device="cuda")
    if c.get("owner", -1) >= 0:
        sure[c["owner"]] = True
    if reliable is not None:
        sure |= reliable.bool()
    if c["loss"] == "bernoulli":
        arrived = (w0 >= _threshold(c["p"])) | sure
    else:
        to_bad, to_good = ((w0 < _threshold(c[k])).cpu().numpy() for k in ("p_gb", "p_bg"))
        bad = np.zeros(n, bool)
        path = np.zeros((n, P), bool)
        for k in range(P):
            bad = np.where(bad, ~to_good[:, k], to_bad[:, k])
            path[:, k] = bad
        state = torch.from_numpy(bad.astype(np.uint8))
        at = torch.from_numpy(path).cuda()
        thr = torch.where(at, _threshold(c["loss_bad"]), _threshold(c["loss_good"]))
        arrived = (w1 >= thr) | sure
    g = c.get("parity", 0)
    if g:
        groups = -(-P // g)
        lost = torch.zeros((n, groups * g), dtype=torch.bool, device="cuda")
        lost[:, :P] = ~arrived
        lost = lost.view(n, groups, g)
        par = _words(n, groups, step, direction + 2, seed)[0] >= _threshold(c["p"])
        rebuilt = (lost.sum(2) == 1) & par
        arrived = ~(lost & ~rebuilt[..., None]).reshape(n, -1)[:, :P]
    return arrived, state.cuda()


def _packet_arrival(c, step, reliable):
    """Arrival probability of each packet of a lossy row, [P] in 64 bits."""
    P = _packets(c)
    q = torch.full((P,), 1.0 - c.get("p", 0.0), dtype=torch.float64, device="cuda")
    if c["loss"] != "bernoulli":
        moves = torch.arange(P, dtype=torch.float64, device="cuda") + float(step) * P + 1.0
        s = c["p_gb"] + c["p_bg"]
        bad = (c["p_gb"] / s) * (1.0 - (1.0 - s) ** moves)
        q = 1.0 - (bad * c["loss_bad"] + (1.0 - bad) * c["loss_good"])
    elif c["parity"]:
        g = c["parity"]
        k = torch.arange(P, device="cuda")
        size = torch.minimum((k // g + 1) * g, torch.tensor(P, device="cuda")) - k // g * g
        rel = torch.zeros(-(-P // g) * g, device="cuda", dtype=torch.long)
        if reliable is not None:
            rel[:P] = reliable.long()
        others = rel.view(-1, g).sum(1)[k // g] - rel[:P]
        q = q + (1.0 - q) * q ** (size - others).double()
    return q


def _spread(per_packet, c):
    """One value per element from one value per packet."""
    return per_packet.repeat_interleave(c["packet"])[: c["d"]]


def _f32(x):
    return float(np.float32(x))


def _updated(c, step, theta, m, v, g):
    lr = _f32(c["lr"])
    if c["opt"] == "sgd":
        return theta - lr * g, None, None
    if c["opt"] == "momentum":
        m = _f32(c["momentum"]) * m + g
        return theta - lr * m, m, None
    b1, b2, t = _f32(c["beta1"]), _f32(c["beta2"]), step + 1
    m = b1 * m + (1.0 - b1) * g
    v = b2 * v + (1.0 - b2) * g * g
    return theta - lr * (m / (1.0 - b1 ** t)) / ((v / (1.0 - b2 ** t)).sqrt() + _f32(c["eps"])), m, v


def _aggregate(c, grads, arrived, g_prev=None, weight=None, sure_row=-1, sure_packet=None):
    """(g_hat, counts) over arrived rows; g_prev takes what arrived."""
    n, d = c["n"], c["d"]
    total = torch.zeros(d, dtype=torch.float64, device="cuda")
    own = torch.zeros_like(total)
    for i in range(n):
        here = _spread(arrived[i], c)
        x = grads[i, :d].double()
        if g_prev is not None:
            total += torch.where(here, x, g_prev[i, :d].double())
            g_prev[i, :d] = torch.where(here, grads[i, :d], g_prev[i, :d])
        elif i == sure_row:
            own = x
        else:
            total += torch.where(here, x, 0.0)
    counts = arrived.sum(0, dtype=torch.int32)
    if g_prev is not None:
        return total / n, counts
    if weight is not None:
        w = weight.clone()
        if sure_packet is not None:
            w[sure_packet.bool()] = 1.0
        return (total * _spread(w, c) + own) / n, counts
    k = _spread(counts.double(), c)
    return torch.where(k > 0, total / k.clamp(min=1.0), 0.0), counts


def _drift(c, replicas, ref):
    """(max_abs, mean_sq, rms, mean_abs_to_master) of the rows, in 64 bits."""
    n, d = c["n"], c["d"]
    s1, s2 = torch.zeros_like(ref), torch.zeros_like(ref)
    hi, lo = torch.full_like(ref, -math.inf), torch.full_like(ref, math.inf)
    gap = 0.0
    for i in range(n):
        x = replicas[i, :d].double()
        hi, lo = torch.maximum(hi, x), torch.minimum(lo, x)
        x = x - ref
        s1, s2, gap = s1 + x, s2 + x * x, gap + x.abs().sum()
    mean_sq = (n * s2 - s1 * s1).clamp(min=0.0).sum() / (d * max(n * (n - 1) / 2, 1))
    return torch.stack([(hi - lo).max(), mean_sq, mean_sq.sqrt(), gap / (n * d)])


def exact(case, seed):
    c, s = case, prepare(case, seed)
    d, step = c["d"], FIRST_STEP
    theta = s["theta"].double()
    reliable = s.get("reliable")
    if c["kind"] == "update":
        theta, m, v = _updated(c, step, theta, *(s[k] if s[k] is None else s[k].double()
                                                 for k in ("m", "v")), s["g_hat"].double())
        return dict(theta=theta, m=m, v=v)
    if c["kind"] == "drift":
        # the counts are whole numbers, compared between runs
        ref = s["theta"].to(_DTYPE[c["rdtype"]]).double()
        return dict(drift=_drift(c, s["replicas"], ref), drift_counts=None)
    if c["kind"] == "aggregate":
        arrived, state = _masks(c, step, 0, seed, None)
        g, counts = _aggregate(c, s["grads"], arrived)
        return dict(arrived=arrived.byte(), ge_state=state, g_hat=g, counts=counts)
    out = {}
    if c["kind"] == "step":
        arrived, state = _masks(c, step, 0, seed, reliable)
        ht = c["estimator"] == "horvitz_thompson"
        g, counts = _aggregate(
            c, s["grads"], arrived, g_prev=s["g_prev"],
            weight=1.0 / _packet_arrival(c, step, reliable) if ht else None,
            sure_row=c["owner"] if ht else -1, sure_packet=reliable)
        theta, m, v = _updated(c, step, theta, *(s[k] if s[k] is None else s[k].double()
                                                 for k in ("m", "v")), g)
        out = dict(theta=theta, m=m, v=v, ge_g=state, g_prev=s["g_prev"],
                   arrived_g=arrived.byte() if c["masks_out"] else None,
                   counts=counts if c["masks_out"] else None)
    arrived, state = _masks(c, step, 1, seed, reliable)
    ref = theta.float().to(_DTYPE[c["rdtype"]])
    replicas = s["replicas"]
    for i in range(c["n"]):
        replicas[i, :d] = torch.where(_spread(arrived[i], c), ref, replicas[i, :d])
    if c["kind"] == "broadcast":
        return dict(arrived=arrived.byte(), ge_state=state, replicas=replicas)
    out.update(replicas=replicas, ge_b=state, arrived_b=arrived.byte() if c["masks_out"] else None,
               ages=(~arrived).to(torch.int16) if c["ages"] else None)
    if c["drift"]:
        out.update(drift=_drift(c, replicas, ref.double()), drift_counts=None)
    return out
