"""Flat tiles: packet lengths that do not fill the chunks of one packet.

A tile then covers consecutive elements of several packets, with each
thread's elements in up to two (bf16 rows) or four (fp32 rows) of them.  The
lengths here put packet borders inside a thread's vector, at a wavefront's and
a tile's edge, and one packet over many tiles; worker counts cross the 32- and
64-row mask words and the ballots that hold several packets.
"""
import numpy as np
import pytest
import torch

import paper_2507_07114_amd as ll
import workloads as wl

import dispatch_rules as rules
import parity
from test_gpu_fused import _bit_equal, _snapshot, _stagewise
from test_gpu_fuzz import OPTS, test_random_configuration as check_configuration
from test_gpu_pacing import _step, restore_pacing  # noqa: F401

pytestmark = pytest.mark.gpu
DEV = "cuda"

BERN = dict(kind=wl.BERNOULLI, p=0.3)
GE = dict(kind=wl.GILBERT_ELLIOTT, p_gb=0.2, p_bg=0.3, loss_good=0.05, loss_bad=0.7)


def _case(case, n, packet, d, gdtype, opt, loss=BERN, est="arrived_mean", owner=-1,
          reliable=False, parity=0, lam=0.0, flat=True):
    return dict(case=case, n=n, packet=packet, d=d, gdtype=gdtype, opt=opt, loss=loss, est=est,
                owner=owner, reliable=reliable, parity=parity, lam=lam, flat=flat)


def _tiling(w, rdtype=None, step=True):
    """Whether a workload's step and drift pass (step=False: an aggregate or a
    broadcast of such rows by itself) run on flat tiles."""
    return rules.tiles((rdtype or w.gdtype) == wl.F32, w.n, w.d, w.packet, step)[1] > 0


CASES = [
    # the shortest flat packets (33 per tile), and the longest that are not
    _case(2000, 3, 64, 70_001, wl.BF16, "adam"),
    _case(2001, 3, 63, 4_001, wl.BF16, "adam", flat=False),
    _case(2002, 1, 65, 2_048, wl.F32, "sgd", flat=False),
    # Ethernet payloads; owner, reliable and parity packets; empty packets
    _case(2003, 16, 750, 20_011, wl.BF16, "adam", owner=5, reliable=True, parity=4),
    _case(2004, 33, 375, 10_007, wl.F32, "momentum",
          dict(kind=wl.BERNOULLI, p=0.97), lam=0.1, flat=False),
    _case(2005, 2, 2250, 4_096, wl.BF16, "sgd", dict(kind=wl.BERNOULLI, p=1.0), lam=0.1),
    # Horvitz-Thompson: weights that differ between the packets of a tile
    _case(2006, 20, 100, 6_001, wl.BF16, "adam", est="horvitz_thompson", owner=19, reliable=True,
          parity=3),
    _case(2007, 70, 333, 6_002, wl.F32, "momentum", GE, est="horvitz_thompson", owner=66,
          reliable=True, flat=False),
    # stale fill: a vector half from the arrived row, half from the last one
    _case(2008, 31, 750, 12_345, wl.BF16, "momentum", est="stale_fill"),
    _case(2009, 65, 129, 5_003, wl.F32, "sgd", GE, est="stale_fill", reliable=True, flat=False),
    # one element more and less than a tile, and a packet of several tiles
    _case(2010, 8, 2047, 16_384, wl.BF16, "adam"),
    _case(2011, 64, 1025, 16_385, wl.F32, "adam", GE),
    _case(2012, 130, 8191, 30_001, wl.BF16, "adam"),
    _case(2013, 1024, 204, 3_000, wl.F32, "adam", owner=1000, flat=False),
    # the fp32 cases above run on chunk tiles, being so few; the same on flat ones
    _case(2020, 1, 65, 83_000, wl.F32, "sgd"),
    _case(2021, 33, 375, 50_011, wl.F32, "momentum",
          dict(kind=wl.BERNOULLI, p=0.97), lam=0.1),
    _case(2022, 70, 333, 50_002, wl.F32, "momentum", GE, est="horvitz_thompson", owner=66,
          reliable=True),
    _case(2023, 65, 129, 50_003, wl.F32, "sgd", GE, est="stale_fill", reliable=True),
    _case(2024, 1024, 521, 3_000, wl.F32, "adam", owner=1000),
    # lengths a multiple of 8, flat from 1025 (bf16) or 4097 (fp32) chunk tiles
    # on and chunks up to there
    _case(2014, 9, 256, 256 * 1025 - 200, wl.BF16, "adam"),
    _case(2015, 9, 256, 256 * 1024, wl.BF16, "adam", flat=False),
    _case(2016, 2, 72, 72 * 4097 - 5, wl.F32, "momentum", est="stale_fill"),
    # off the 128-byte lines, but in few tiles
    _case(2017, 12, 6000, 400_001, wl.BF16, "sgd", flat=False),
]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: f"case{c['case']}")
def test_flat_step_matches_the_oracle(cfg):
    f32 = cfg["gdtype"] == wl.F32
    assert (rules.tiles(f32, cfg["n"], cfg["d"], cfg["packet"])[1] > 0) == cfg["flat"]
    check_configuration(cfg)


# tiles: (of the step and the drift pass, of the aggregate and the broadcast), flat?
@pytest.mark.parametrize("name,n,d,L,pad,tiles", [
    ("n8_d16m_bf16_adam", 8, 40_961, 750, 0, (True, True)),
    ("n8_d16m_bf16_adam", 200, 9_001, 250, 8, (True, True)),
    ("n64_d48m_f32_sgd_drift", 64, 20_005, 375, 4, (False, False)),
    ("n64_d48m_f32_sgd_drift", 64, 50_005, 375, 4, (True, True)),
    ("n16_d256m_f32_ge_momentum", 17, 30_720, 2250, 0, (True, True)),
    # full chunks off the 128-byte lines: few rows of a step stay with chunks,
    # stages by themselves do not, and with more rows all are flat
    ("n8_d16m_bf16_adam", 8, 1_200_000, 1928, 0, (False, False)),
    ("n8_d16m_bf16_adam", 8, 2_000_003, 1928, 0, (False, True)),
    ("n8_d16m_bf16_adam", 11, 2_060_001, 6000, 0, (False, True)),
    ("n8_d16m_bf16_adam", 12, 2_060_001, 6000, 0, (True, True)),
])
def test_flat_step_equals_stagewise(name, n, d, L, pad, tiles):
    w = wl.scaled(wl.WORKLOADS[name], n=n, d=d, packet=L)
    assert (_tiling(w), _tiling(w, step=False)) == tiles
    a, b = parity.DeviceState(w, pad=pad), parity.DeviceState(w, pad=pad)
    for t in range(2):
        print(f"flat {name} n={n} d={d} L={L} step {t}", flush=True)
        wl.draw_grads(w, t, device=DEV, ld=a.ld, out=a.grads)
        b.grads.copy_(a.grads)
        a.fused(t)
        _stagewise(b, t)
        sa, sb = _snapshot(a), _snapshot(b)
        sa["drift"]["empty_packets"] = sb["drift"]["empty_packets"] = 0
        assert sa["drift"] == sb["drift"], (sa["drift"], sb["drift"])
        for k in sa:
            if k != "drift":
                assert _bit_equal(sa[k], sb[k]), f"step {t}: {k} differs"


def _with_replicas(w, rdtype):
    """Two states of a workload whose replica rows are of type rdtype."""
    out = parity.DeviceState(w), parity.DeviceState(w)
    for dev in out:
        dev.replicas = torch.zeros((w.n, dev.ld), dtype=wl.torch_dtype(rdtype), device=DEV)
        dev.replicas[:, : w.d] = dev.theta.to(dev.replicas.dtype)[None, :]
    return out


@pytest.mark.parametrize("name,n,d,L,rdtype", [
    ("n64_llama7b_shard_bf16_adam", 64, 2048 * 2600 + 1009, 750, wl.BF16),
    ("n64_d48m_f32_sgd_drift", 40, 1024 * 5000 + 13, 1500, wl.F32),
    # rows of unlike types
    ("n64_llama7b_shard_bf16_adam", 33, 1024 * 2600 + 77, 750, wl.F32),
    ("n64_d48m_f32_sgd_drift", 33, 2048 * 2600 + 501, 333, wl.BF16),
])
@pytest.mark.parametrize("masks_out,drift", [(True, True), (False, False)])
def test_flat_paced_step_is_bit_identical_to_unpaced(name, n, d, L, rdtype, masks_out, drift,
                                                     restore_pacing):  # noqa: F811
    w = wl.scaled(wl.WORKLOADS[name], n=n, d=d, packet=L)
    assert _tiling(w, rdtype)
    a, b = _with_replicas(w, rdtype)
    for t in range(2):
        print(f"flat paced {name} n={n} L={L} {rdtype} step {t}", flush=True)
        wl.draw_grads(w, t, device=DEV, ld=a.ld, out=a.grads)
        b.grads.copy_(a.grads)
        ll.ll_set_pacing("always")
        _step(a, t, masks_out=masks_out, drift=drift, workspace=True)
        ll.ll_set_pacing("never")
        _step(b, t, masks_out=masks_out, drift=drift, workspace=True)
        sa, sb = _snapshot(a), _snapshot(b)
        assert not drift or sa["drift"] == sb["drift"], (sa["drift"], sb["drift"])
        for k in sa:
            if k != "drift" and (masks_out or not k.startswith("arrived")):
                assert _bit_equal(sa[k], sb[k]), f"step {t}: {k} differs"


@pytest.mark.parametrize("gdtype,rdtype", [(wl.BF16, wl.F32), (wl.F32, wl.BF16)])
@pytest.mark.parametrize("L", [750, 333])
@pytest.mark.parametrize("est", ["arrived_mean", "horvitz_thompson", "stale_fill"])
def test_flat_step_of_unlike_row_types_equals_stagewise(est, L, gdtype, rdtype):
    """The step takes the replicas' tiles for both rows, each stage its own
    rows': 8-byte halves of bf16 gradient rows and unsplit fp32 ones."""
    n, d = 20, 83_005
    w = wl.scaled(wl.WORKLOADS["n8_d16m_bf16_adam"], n=n, d=d, packet=L, gdtype=gdtype,
                  loss=dict(kind=wl.BERNOULLI, p=0.3))
    assert _tiling(w, rdtype) and _tiling(w, gdtype, step=False)
    a, b = _with_replicas(w, rdtype)
    P, spec = w.num_packets, parity.loss_spec(w)
    prev = [torch.randn(a.grads.shape, generator=torch.Generator(DEV).manual_seed(1), device=DEV)
            .to(a.grads.dtype) for _ in range(2)]
    owner = 3 if est == "horvitz_thompson" else -1
    ext = [ll.ext(est, owner=owner, g_prev=g if est == "stale_fill" else None,
                  arrival_prob=0.7 if est == "horvitz_thompson" else 0.0) for g in prev]
    for t in range(2):
        print(f"flat unlike {est} {gdtype}/{rdtype} L={L} step {t}", flush=True)
        wl.draw_grads(w, t, device=DEV, ld=a.ld, out=a.grads)
        b.grads.copy_(a.grads)
        a.fused(t, ext=ext[0])
        g_hat = torch.empty(d, device=DEV)
        only = ll.ext(owner=owner)
        ll.ll_masks(n, P, t, ll.LL_DIR_GRAD, spec, b.arrived_g, ext=only)
        ll.lossy_aggregate(b.grads, b.arrived_g, d=d, packet=L, g_hat=g_hat, counts=b.counts,
                           theta=b.theta, ext=ext[1])
        ll.shard_step(parity.opt_spec(w), t, b.theta, g_hat, m=b.m, v=b.v)
        ll.ll_masks(n, P, t, ll.LL_DIR_BCAST, spec, b.arrived_b, ext=only)
        ll.lossy_broadcast(b.theta, b.replicas, b.arrived_b, d=d, packet=L)
        ll.drift_stats(b.replicas, d=d, packet=L, workspace=b.workspace, out=b.drift,
                       theta=b.theta, arrived_bc=b.arrived_b)
        sa, sb = _snapshot(a), _snapshot(b)
        sa["drift"]["empty_packets"] = sb["drift"]["empty_packets"] = 0
        assert sa["drift"] == sb["drift"], (sa["drift"], sb["drift"])
        for k in sa:
            if k != "drift":
                assert _bit_equal(sa[k], sb[k]), f"step {t}: {k} differs"
        assert _bit_equal(prev[0], prev[1]), f"step {t}: g_prev differs"


@pytest.mark.parametrize("gdtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("est", ["arrived_mean", "horvitz_thompson", "stale_fill"])
@pytest.mark.parametrize("d", [10_007, 50_007])  # fp32 rows: chunk tiles, flat ones
def test_flat_aggregate_stage(est, gdtype, d):
    """lossy_aggregate alone: lost elements hold NaN and are never used."""
    n, L = 37, 333
    f32 = gdtype == torch.float32
    assert (rules.tiles(f32, n, d, L, step=False)[1] > 0) == (d > 50_000 or not f32)
    P = -(-d // L)
    gen = torch.Generator(device=DEV).manual_seed(7)
    arrived = (torch.rand((n, P), generator=gen, device=DEV) < 0.6).to(torch.uint8)
    arrived[:, 3] = 0
    reliable = torch.zeros(P, dtype=torch.uint8, device=DEV)
    reliable[5::7] = 1
    arrived[:, 5::7] = 1
    arrived[2] = 1
    owner = 2 if est == "horvitz_thompson" else -1
    if owner < 0:
        arrived[2, 3] = 0
    ld = -(-d // 8) * 8
    here = arrived.bool().repeat_interleave(L, 1)[:, :d]
    g = torch.full((n, ld), float("nan"), device=DEV, dtype=gdtype)
    vals = torch.randn((n, d), generator=gen, device=DEV).to(gdtype)
    g[:, :d] = torch.where(here, vals, g[:, :d])
    prev0 = torch.randn((n, ld), generator=gen, device=DEV).to(gdtype)
    prev = prev0.clone() if est == "stale_fill" else None
    theta = torch.randn(d, generator=gen, device=DEV)
    g_hat = torch.zeros(d, device=DEV)
    counts = torch.zeros(P, dtype=torch.int32, device=DEV)
    e = ll.ext(est, owner=owner, reliable=reliable, g_prev=prev,
               arrival_prob=0.6 if est == "horvitz_thompson" else 0.0)
    lam = 0.25 if est == "arrived_mean" else 0.0
    ll.lossy_aggregate(g, arrived, d=d, packet=L, g_hat=g_hat, counts=counts, ext=e,
                       fallback_lambda=lam, theta=theta)
    torch.cuda.synchronize()
    x = torch.where(here, vals.double(), 0.0)
    K = arrived.sum(0, dtype=torch.int32)
    assert torch.equal(counts, K)
    k = K.repeat_interleave(L)[:d].double()
    if est == "arrived_mean":
        want = torch.where(k > 0, x.sum(0) / k.clamp(min=1), lam * theta.double())
    elif est == "horvitz_thompson":
        sure = reliable.bool().repeat_interleave(L)[:d]
        w = np.float32(1.0 / 0.6).item()
        wt = torch.where(sure, 1.0, torch.tensor(w, dtype=torch.float64, device=DEV))
        lossy = x.clone()
        lossy[owner] = 0
        want = (lossy.sum(0) * wt + x[owner]) / n
    else:
        mix = torch.where(here, vals, prev0[:, :d])
        want = mix.double().sum(0) / n
        assert torch.equal(prev[:, :d], mix) and torch.equal(prev[:, d:], prev0[:, d:])
    # a sequential fp32 sum of n terms of either sign and two more roundings
    tol = 1e-5 * x.abs().sum(0).clamp(min=1.0)
    assert ((g_hat.double() - want).abs() <= tol).all()


@pytest.mark.parametrize("gdtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("p", [0.5, 1.0])
def test_flat_drift_skips_nonfinite_elements_that_arrived(gdtype, p):
    """A master value that is infinite, NaN or overflows the replica type adds
    nothing to the drift where every row holds it, also beside an element of a
    lossy packet in the same vector: such a row's drift is that of the other
    elements."""
    n, d, L = 5, 50_003, 333  # whole tiles and a ragged end
    assert rules.tiles(gdtype == torch.float32, n, d, L)[1] > 0
    P = -(-d // L)
    print(f"flat nonfinite {gdtype} p={p}", flush=True)
    gen = torch.Generator(device=DEV).manual_seed(3)
    sure = torch.zeros(P, dtype=torch.uint8, device=DEV)
    sure[::2] = 1
    on_sure = sure.bool().repeat_interleave(L)[:d]
    ld = -(-d // 8) * 8
    theta = torch.randn(d, generator=gen, device=DEV)
    replicas = torch.zeros((n, ld), dtype=gdtype, device=DEV)
    replicas[:, :d] = (theta + 0.1 * torch.randn((n, d), generator=gen, device=DEV)).to(gdtype)
    at = torch.arange(d, device=DEV) % L
    edge = on_sure & ((at < 4) | (at >= L - 4))
    odd = torch.tensor([float("inf"), float("-inf"), float("nan"), 3.4e38], device=DEV)
    theta[edge] = odd[torch.arange(int(edge.sum()), device=DEV) % 4]
    drift = ll.drift_buffer()
    ws = torch.zeros(ll.ll_workspace_bytes(n, d, L), dtype=torch.uint8, device=DEV)
    loss = ll.bernoulli(p, seed=5)
    ll.lossy_step_fused(d=d, packet=L, step=0, loss_g=loss, loss_b=loss,
                        grads=torch.zeros((n, ld), dtype=gdtype, device=DEV), opt=ll.sgd(0.0),
                        theta=theta, replicas=replicas, workspace=ws, drift=drift,
                        ext=ll.ext(reliable=sure))
    got = ll.read_drift(drift)
    rest, ref = replicas.clone(), theta.clone()
    rest[:, :d][:, on_sure] = 0
    ref[on_sure] = 0
    want = parity.torch_drift(rest, ref, d)
    assert want["mean_abs_to_master"] > 0
    parity.check_drift_close(got, want, f"{gdtype} p={p}")


def test_stale_fill_without_drift_equals_the_step_with_it():
    """On both sides of a rule: the step without drift on chunk tiles, the step
    with drift on flat ones."""
    n, L, d = 18, 256, 256 * 1500 - 3
    print(f"stale fill on both tilings n={n} d={d}", flush=True)
    assert rules.tiles(False, n, d, L, fill_only=True)[1] == 0 < rules.tiles(False, n, d, L)[1]
    gen = torch.Generator(device=DEV).manual_seed(4)
    rows = [torch.randn((n, -(-d // 8) * 8), generator=gen, device=DEV).bfloat16()
            for _ in range(3)]
    vecs = [torch.randn(d, generator=gen, device=DEV) for _ in range(2)]
    loss, opt = ll.bernoulli(0.3, seed=9), ll.sgd_momentum(0.01, 0.9)
    ws = torch.zeros(ll.ll_workspace_bytes(n, d, L), dtype=torch.uint8, device=DEV)
    out = []
    for drift in (None, ll.drift_buffer()):
        (grads, prev, reps), (theta, m) = [x.clone() for x in rows], [x.clone() for x in vecs]
        ll.lossy_step_fused(d=d, packet=L, step=2, loss_g=loss, loss_b=loss, grads=grads, opt=opt,
                            theta=theta, replicas=reps, m=m, workspace=ws, drift=drift,
                            ext=ll.ext("stale_fill", g_prev=prev))
        out.append((grads, prev, reps, theta, m))
    for name, x, y in zip(("grads", "g_prev", "replicas", "theta", "m"), *out):
        assert _bit_equal(x, y), name
