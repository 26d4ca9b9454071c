"""The paced broadcast (row stores wait for clock slots scaled by the sampled
share of arrived rows) is bit-identical to the unpaced one, kept and far too
fast, on chunk and flat tiles, with everything, nothing and some rows arrived,
and from a graph.  The aggregate and drift calls beside it read no pacing
setting; they check that a paced broadcast leaves its neighbours alone."""
import pytest
import torch

import paper_2507_07114_amd as ll

from test_gpu_pacing import restore_pacing  # noqa: F401

pytestmark = pytest.mark.gpu
DEV = "cuda"

SCHEDULES = [
    dict(),
    dict(bytes_per_s=5.0e14, bytes_per_s_f32=5.0e14),
    dict(overlap=2, resident=2),
]


def _stages(g, reps, theta, arrived, d, L, lam):
    n, P = arrived.shape
    g_hat = torch.zeros(d, device=DEV)
    counts = torch.zeros(P, dtype=torch.int32, device=DEV)
    out = reps.clone()
    ws = torch.zeros(ll.ll_workspace_bytes(n, d, L), dtype=torch.uint8, device=DEV)
    drift, bare = ll.drift_buffer(), ll.drift_buffer()
    ll.lossy_aggregate(g, arrived, d=d, packet=L, g_hat=g_hat, counts=counts,
                       fallback_lambda=lam, theta=theta)
    ll.lossy_broadcast(theta, out, arrived, d=d, packet=L)
    ll.drift_stats(out, d=d, packet=L, workspace=ws, out=drift, theta=theta, arrived_bc=arrived)
    ll.drift_stats(out, d=d, packet=L, workspace=ws, out=bare)
    torch.cuda.synchronize()
    return [x.view(torch.uint8).cpu() for x in (g_hat, counts, out, drift, bare)]


@pytest.mark.parametrize("sched", range(len(SCHEDULES)))
@pytest.mark.parametrize("p", [0.0, 0.2, 1.0])
@pytest.mark.parametrize("n,d,L,dtype", [
    (3, 5_000, 1024, torch.float32),             # fewer tiles than a round
    (20, 2048 * 2300 + 8, 4096, torch.bfloat16),
    (20, 2048 * 2300 + 3, 750, torch.bfloat16),  # flat tiles
    (70, 1024 * 2100 + 5, 3000, torch.float32),  # 2151 chunk tiles, few enough
    (70, 1024 * 2100 + 5, 1300, torch.float32),  # flat tiles
])
def test_paced_stages_are_bit_identical(n, d, L, dtype, p, sched, restore_pacing):  # noqa: F811
    print(f"paced stages n={n} d={d} L={L} {dtype} p={p} schedule {sched}", flush=True)
    gen = torch.Generator(device=DEV).manual_seed(n + d)
    P, ld = -(-d // L), -(-d // 8) * 8
    arrived = (torch.rand((n, P), generator=gen, device=DEV) >= p).to(torch.uint8)
    g = torch.randn((n, ld), generator=gen, device=DEV).to(dtype)
    reps = torch.randn((n, ld), generator=gen, device=DEV).to(dtype)
    theta = torch.randn(d, generator=gen, device=DEV)
    ll.ll_set_pacing("never")
    want = _stages(g, reps, theta, arrived, d, L, 0.5)
    ll.ll_set_pacing("always", **SCHEDULES[sched])
    for _ in range(2):
        got = _stages(g, reps, theta, arrived, d, L, 0.5)
        for name, a, b in zip(("g_hat", "counts", "replicas", "drift", "drift of rows alone"),
                              got, want):
            assert torch.equal(a, b), name


@pytest.mark.parametrize("n,d,L,dtype", [
    (20, 2048 * 2300 + 8, 4096, torch.bfloat16),
    (40, 1024 * 2100 + 5, 750, torch.float32),  # flat tiles
])
def test_captured_paced_broadcast_replays_like_eager(n, d, L, dtype, restore_pacing):  # noqa: F811
    print(f"captured broadcast n={n} d={d} L={L} {dtype}", flush=True)
    gen = torch.Generator(device=DEV).manual_seed(d)
    P, ld = -(-d // L), -(-d // 8) * 8
    arrived = (torch.rand((n, P), generator=gen, device=DEV) >= 0.3).to(torch.uint8)
    theta = torch.randn(d, generator=gen, device=DEV)
    start = torch.randn((n, ld), generator=gen, device=DEV).to(dtype)
    a, b = start.clone(), start.clone()
    ll.ll_set_pacing("always")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        ll.lossy_broadcast(theta, b, arrived, d=d, packet=L)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ll.lossy_broadcast(theta, b, arrived, d=d, packet=L)
    ll.ll_set_pacing("never")
    for rep in range(3):
        theta.normal_(generator=gen)
        arrived.copy_(torch.rand((n, P), generator=gen, device=DEV) >= 0.3)
        a.copy_(start)
        b.copy_(start)
        ll.lossy_broadcast(theta, a, arrived, d=d, packet=L)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), f"replay {rep} differs"
