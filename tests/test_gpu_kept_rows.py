"""Small calls load their rows with the plain cache policy (kept rows), others
past the caches: the same call on one shard and on slices of it, which have too
few tiles to keep their rows, gives the same bits."""
import pytest
import torch

import paper_2507_07114_amd as ll

import dispatch_rules as rules

pytestmark = pytest.mark.gpu
DEV = "cuda"
F32, BF16 = torch.float32, torch.bfloat16


def _bits(x):
    return x.contiguous().view(torch.uint8)


@pytest.mark.parametrize("d,L,gd,rd,est", [
    (2048 * 1030 + 5, 4096, BF16, BF16, "arrived_mean"),      # chunk tiles, ragged end
    (2048 * 1026 + 3, 750, BF16, BF16, "arrived_mean"),       # flat tiles
    (1024 * 1030 + 5, 2048, F32, F32, "horvitz_thompson"),
    (1024 * 1030 + 1, 333, F32, F32, "stale_fill"),
    (2048 * 1030 + 5, 4096, BF16, BF16, "stale_fill"),
    (2048 * 1026 + 3, 750, BF16, BF16, "stale_fill"),
    (1024 * 1030 + 8, 2048, BF16, F32, "arrived_mean"),       # rows of unlike types
    (1024 * 1030 + 3, 750, BF16, F32, "horvitz_thompson"),
    (2048 * 1030 + 8, 4096, F32, BF16, "stale_fill"),
    (2048 * 1026 + 3, 750, F32, BF16, "arrived_mean"),
])
def test_kept_rows_equal_streamed_ones(d, L, gd, rd, est):
    n, P, ld = 3, -(-d // L), -(-d // 8) * 8
    print(f"kept rows d={d} L={L} grads {gd} replicas {rd} {est}", flush=True)
    cut = d // 6 // (8 * L) * (8 * L)  # slices start on packets and on 16 bytes
    parts = [(i * cut, d if i == 5 else (i + 1) * cut) for i in range(6)]
    fill = est == "stale_fill"
    moved = n * d * (gd.itemsize * (2 if fill else 1) + rd.itemsize) + 12 * d
    assert rules.keeps(rules.tiles(rd == F32, n, d, L)[0], moved, fill=fill)
    for a, b in parts:
        assert not rules.keeps(rules.tiles(gd == F32, n, b - a, L, False)[0], moved, fill=fill)
        assert not rules.keeps(rules.tiles(rd == F32, n, b - a, L)[0], moved, drift=True)
    gen = torch.Generator(device=DEV).manual_seed(L + d)
    grads, prev = (torch.randn((n, ld), generator=gen, device=DEV).to(gd) for _ in range(2))
    start = torch.randn((n, ld), generator=gen, device=DEV).to(rd)
    theta0, m0 = (torch.randn(d, generator=gen, device=DEV) for _ in range(2))
    v0 = torch.rand(d, generator=gen, device=DEV)
    ws = torch.zeros(ll.ll_workspace_bytes(n, d, L), dtype=torch.uint8, device=DEV)
    opt, loss = ll.adam(3e-4, 0.9, 0.95, 1e-8), ll.bernoulli(0.4, seed=5)

    def variant(g_prev):
        if est == "stale_fill":
            return ll.ext(est, g_prev=g_prev)
        return ll.ext(est, arrival_prob=0.6) if est == "horvitz_thompson" else None

    theta, m, v, reps, g_prev = (x.clone() for x in (theta0, m0, v0, start, prev))
    arrived = [torch.zeros((n, P), dtype=torch.uint8, device=DEV) for _ in range(2)]
    drift = ll.drift_buffer()
    ll.lossy_step_fused(d=d, packet=L, step=3, loss_g=loss, loss_b=loss, grads=grads, opt=opt,
                        theta=theta, replicas=reps, m=m, v=v, arrived_g=arrived[0],
                        arrived_b=arrived[1], workspace=ws, drift=drift, ext=variant(g_prev))
    alone_prev, alone = prev.clone(), torch.zeros(d, device=DEV)
    ll.lossy_aggregate(grads, arrived[0], d=d, packet=L, g_hat=alone, ext=variant(alone_prev))
    pass_drift = ll.drift_buffer()
    ll.drift_stats(reps, d=d, packet=L, workspace=ws, out=pass_drift, theta=theta,
                   arrived_bc=arrived[1])

    w_th, w_m, w_v, w_reps, w_prev = (x.clone() for x in (theta0, m0, v0, start, prev))
    g_hat = torch.zeros(d, device=DEV)
    drifts = []
    for a, b in parts:
        mg, mb = (x[:, a // L: -(-b // L)].contiguous() for x in arrived)
        kw = dict(d=b - a, packet=L)
        ll.lossy_aggregate(grads[:, a:b], mg, g_hat=g_hat[a:b], ext=variant(w_prev[:, a:b]), **kw)
        ll.shard_step(opt, 3, w_th[a:b], g_hat[a:b], m=w_m[a:b], v=w_v[a:b])
        ll.lossy_broadcast(w_th[a:b], w_reps[:, a:b], mb, **kw)
        out = ll.drift_buffer()
        ll.drift_stats(w_reps[:, a:b], workspace=ws, out=out, theta=w_th[a:b], arrived_bc=mb, **kw)
        drifts.append((b - a, ll.read_drift(out)))
    for name, x, y in (("theta", theta, w_th), ("m", m, w_m), ("v", v, w_v),
                       ("replicas", reps, w_reps), ("aggregate", alone, g_hat)):
        assert torch.equal(_bits(x), _bits(y)), name
    if fill:
        assert torch.equal(_bits(g_prev), _bits(w_prev))
        assert torch.equal(_bits(alone_prev), _bits(w_prev))
    got, by_pass = ll.read_drift(drift), ll.read_drift(pass_drift)
    assert {**got, "empty_packets": 0} == {**by_pass, "empty_packets": 0}
    assert got["max_abs"] == max(r["max_abs"] for _, r in drifts)
    assert got["stale_packets"] == sum(r["stale_packets"] for _, r in drifts)
    # fp64 sums over the same per-element terms in another order
    for k in ("mean_sq", "mean_abs_to_master"):
        want = sum(e * r[k] for e, r in drifts) / d
        assert abs(got[k] - want) <= 1e-12 * abs(want), k
