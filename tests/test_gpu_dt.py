"""GPU parity of delta-tracking path tracing over bricks.

Routing is bit-exact: per forward step, the counts per domain and every
queued item's position, direction, path id, random stream, draw count,
scattering count and kind equal the oracle's. Weights and contributions are
float32 on the GPU and float64 in the oracle: within 1e-5 relative."""
import numpy as np
import pytest
import torch

from gpu_util import announce, device, rel_close
from paper_2605_30294_amd import rafi
from paper_2605_30294_amd import workloads as W

pytestmark = pytest.mark.gpu

RTOL = 1e-5
ATOL = 1e-30


def _stepwise(vol_np, grid, views, kappa, smax, albedo, light, radiance, B, seed):
    dev = device()
    nv, w, h = len(views), int(views[0]["width"]), int(views[0]["height"])
    n_paths = nv * w * h
    ctx = rafi.Context(int(np.prod(grid)), rafi.DT_ITEM_BYTES, rafi.dt_capacity(n_paths, B), debug=True)
    vol = torch.from_numpy(vol_np).to(dev)
    vdev = rafi.views_to_device(views, dev)
    contrib = torch.full((n_paths, B), -1.0, dtype=torch.float32, device=dev)
    counters = torch.zeros(2, dtype=torch.int64, device=dev)
    job = rafi.dt_job(vol, grid, vdev, nv, w, h, contrib, None, kappa, smax, albedo, light, radiance, B, seed,
                      counters)
    rafi.dt_raygen(ctx, job)
    counts, queues = [], []
    while True:
        cnt, total, rc = ctx.round()
        q, _ = ctx.copy_queue()
        counts.append(cnt)
        queues.append(q.cpu().numpy().view(np.uint32).reshape(-1, 12).copy())
        if total == 0:
            break
        rafi.dt_trace(ctx, job)
    torch.cuda.synchronize()
    st = ctx.stats()
    ctx.close()
    return dict(contrib=contrib.cpu().numpy(), counts=np.array(counts), queue=np.concatenate(queues), stats=st,
                counters=counters.cpu().numpy())


def _compare(g, o):
    assert np.array_equal(g["counts"], o["round_counts"])
    gq, oq = g["queue"], o["queue"]
    assert gq.shape[0] == oq.shape[0]
    # words: p(3) d(3) w path stream count bounce kind; the oracle logs all but w
    assert np.array_equal(gq[:, [0, 1, 2, 3, 4, 5, 7, 8, 9, 10, 11]], oq)
    ok, i, r = rel_close(gq[:, 6].view(np.float32), o["weights"], RTOL, ATOL)
    assert ok, f"weight of queued item {i}: gpu {gq[i, 6].view(np.float32)} oracle {o['weights'][i]} ({r:.3g} x tol)"
    ok, i, r = rel_close(g["contrib"].ravel(), o["contrib"].ravel(), RTOL, ATOL)
    assert ok, f"contribution {i}: gpu {g['contrib'].ravel()[i]} oracle {o['contrib'].ravel()[i]}"
    assert g["stats"]["bad_dest"] == 0 and g["stats"]["dropped"] == 0


CASES = [
    # n, grid, views, kappa, smax factor, albedo, light, radiance, bounces, seed
    (32, (2, 2, 2), "plusz", 0.05, 1.25, 0.8, (0.0, 0.0, -1.0), 1.0, 4, 1),
    (32, (4, 2, 1), "rot2", 0.08, 1.0, 0.9, (0.6, 0.0, 0.8), 2.0, 3, 2),
    (48, (3, 3, 1), "rot2", 0.04, 2.0, 0.5, (0.0, 0.8, -0.6), 1.5, 2, 3),
    (16, (1, 1, 1), "rot2", 0.2, 1.1, 1.0, (0.0, 0.0, 1.0), 1.0, 5, 4),
]


def _views(kind, n):
    if kind == "plusz":
        return W.plusz_view(n, 40, 40)
    return W.random_views(2, n, 28, 28, seed=50 + n)


@pytest.mark.parametrize("case", CASES)
def test_matches_oracle(orc, case):
    n, grid, vk, kappa, sf, albedo, light, radiance, B, seed = case
    vol = W.blob_volume(n, 40 + seed)
    views = _views(vk, n)
    smax = float(np.float32(kappa * float(vol.max()) * sf))
    announce(f"dt n={n} grid={grid} B={B}")
    g = _stepwise(vol, grid, views, kappa, smax, albedo, light, radiance, B, seed)
    o = orc.dt_render(vol, grid, views, kappa, smax, albedo, light, radiance, B, seed, queue_cap=1 << 22)
    _compare(g, o)
    # every queued item is one tentative point or more; collisions counted once
    assert g["counters"][0] >= g["counts"].sum() and g["counters"][1] <= g["counters"][0]


@pytest.mark.parametrize("n,grid,nv,w,B,scale", [
    (32, (2, 2, 2), 1, 640, 3, 1.0),          # launches over 160 K items, one lane each, and under
    (24, (3, 1, 2), 2, 370, 2, 1.0),
    (24, (2, 1, 1), 1, 40, 2, 1e-13),         # a majorant outside the corrected division's range
    (64, (1, 1, 1), 1, 33, 2, 1.0),           # one brick: visits of up to several hundred points
])
def test_launch_sizes_and_majorants(orc, n, grid, nv, w, B, scale):
    """Both sides of the sizes the launches choose by, one to several hundred
    points per visit, and a majorant too small for the corrected division."""
    vol = W.blob_volume(n, 60 + n, n_blobs=12)
    views = W.random_views(nv, n, w, w, seed=61)
    kappa = 0.3 * scale
    smax = float(np.float32(kappa * float(vol.max()) * (4.0 if n == 64 else 1.1)))
    announce(f"dt n={n} grid={grid} paths={nv * w * w} smax={smax}")
    g = _stepwise(vol, grid, views, kappa, smax, 0.7, (0.6, 0.0, 0.8), 1.0, B, 9)
    o = orc.dt_render(vol, grid, views, kappa, smax, 0.7, (0.6, 0.0, 0.8), 1.0, B, 9, queue_cap=1 << 24)
    _compare(g, o)


@pytest.mark.parametrize("w", [24, 420])            # 32 lanes an item, one lane an item
@pytest.mark.parametrize("kappa,smax", [(1e20, 0.3),   # an infinite extinction
                                        (3e8, 0.3)])   # a finite one whose quotient by the majorant overflows
def test_extinction_far_above_the_majorant(orc, w, kappa, smax):
    """A block whose extinction is infinite, or overflows divided by the
    majorant, as the float32 division has it: shadow rays through it weigh an
    infinity of the oracle's sign, never a NaN; the routing is the oracle's.
    The oracle's weights are float64: its value of a weight that overflows in
    float32 is at least the quotient's overflow times the first weight
    (albedo / 4 pi) of the ray."""
    n, grid = 24, (2, 1, 2)
    vol = np.zeros((n, n, n), dtype=np.float32)
    vol[4:16, 6:20, 5:17] = 1e30
    views = W.random_views(1, n, w, w, seed=63)
    announce(f"dt overflow kappa={kappa} w={w}")
    args = (kappa, smax, 0.7, (0.6, 0.0, 0.8), 1.0, 2, 9)
    g = _stepwise(vol, grid, views, *args)
    o = orc.dt_render(vol, grid, views, *args, queue_cap=1 << 24)
    assert np.array_equal(g["counts"], o["round_counts"])
    assert np.array_equal(g["queue"][:, [0, 1, 2, 3, 4, 5, 7, 8, 9, 10, 11]], o["queue"])
    got, want = g["contrib"], o["contrib"]
    assert not np.isnan(want).any() and not np.isnan(got).any()
    over = np.isinf(got)
    assert over.sum() > got.size // 100
    fmax = float(np.finfo(np.float32).max)
    assert np.all(np.abs(want[over]) >= 0.7 ** 2 / (4 * np.pi) * fmax)
    assert np.all(np.abs(want[~over]) <= fmax * (1 + RTOL))
    assert np.array_equal(np.sign(got[over]), np.sign(want[over]))
    ok, i, r = rel_close(got[~over], want[~over], RTOL, ATOL)
    assert ok, (i, r)


def test_render_entry_point_deterministic(orc):
    dev = device()
    n, grid = 64, (4, 4, 4)
    vol_np = W.blob_volume(n, 91)
    views = W.random_views(1, n, 64, 64, seed=92)
    kappa = 0.05
    smax = float(np.float32(kappa * float(vol_np.max())))
    vol = torch.from_numpy(vol_np).to(dev)
    announce("dt render 64^3")
    a = rafi.dt_render(vol, grid, views, kappa, smax, 0.8, (0.0, 0.6, 0.8), 1.0, 4, 7)
    b = rafi.dt_render(vol, grid, views, kappa, smax, 0.8, (0.0, 0.6, 0.8), 1.0, 4, 7)
    torch.cuda.synchronize()
    assert torch.equal(a["contrib"], b["contrib"]) and torch.equal(a["image"], b["image"])
    o = orc.dt_render(vol_np, grid, views, kappa, smax, 0.8, (0.0, 0.6, 0.8), 1.0, 4, 7)
    assert a["rounds"] == o["rounds"]
    ok, i, r = rel_close(a["contrib"].cpu().numpy().ravel(), o["contrib"].ravel(), RTOL, ATOL)
    assert ok, (i, r)
    # image = contributions summed in event order
    c = a["contrib"].cpu().numpy()
    s = np.zeros(c.shape[0], dtype=np.float32)
    for b_ in range(c.shape[1]):
        s = s + c[:, b_]
    assert np.array_equal(a["image"].cpu().numpy(), s)


def test_capacity_is_checked():
    dev = device()
    n, grid = 32, (2, 2, 2)
    vol = torch.from_numpy(W.blob_volume(n, 5)).to(dev)
    views = W.plusz_view(n, 32, 32)
    ctx = rafi.Context(8, rafi.DT_ITEM_BYTES, 32 * 32)          # room for the raygen only
    vdev = rafi.views_to_device(views, dev)
    contrib = torch.zeros((32 * 32, 2), dtype=torch.float32, device=dev)
    job = rafi.dt_job(vol, grid, vdev, 1, 32, 32, contrib, None, 0.05, 1.0, 0.8, (0, 0, -1), 1.0, 2, 1)
    rafi.dt_raygen(ctx, job)
    _, total, _ = ctx.round(counts=False)
    assert total > 0
    with pytest.raises(rafi.RafiError) as e:
        rafi.dt_trace(ctx, job)
    assert e.value.code == rafi.ERR_ARG
    ctx.close()


@pytest.mark.parametrize("B", [1, 2])
def test_render_dense_medium_few_bounces(orc, B):
    """The pipelined render at rafi_dt_capacity's own sizing, 2 paths (B + 1)
    slots, in a dense medium where most paths collide at once: the
    look-ahead launch only bounds the queue length, so it must not refuse a
    queue that fits. Contributions match the oracle."""
    dev = device()
    n, grid = 32, (2, 2, 2)
    vol_np = W.blob_volume(n, 93)
    views = W.plusz_view(n, 48, 48)
    kappa = 0.6
    smax = float(np.float32(kappa * float(vol_np.max()) * 1.05))
    announce(f"dt render dense B={B}")
    r = rafi.dt_render(torch.from_numpy(vol_np).to(dev), grid, views, kappa, smax, 0.95, (0.0, 0.6, 0.8), 1.0, B,
                       11)
    torch.cuda.synchronize()
    st = r["ctx"].stats()
    assert st["dropped"] == 0 and st["bad_dest"] == 0
    o = orc.dt_render(vol_np, grid, views, kappa, smax, 0.95, (0.0, 0.6, 0.8), 1.0, B, 11)
    assert r["rounds"] == o["rounds"]
    # with two bounces the queue exceeds a quarter of the capacity in some
    # round, where a launch sized for twice the split slots would not fit
    if B == 2:
        assert int(o["round_counts"].sum(axis=1).max()) > rafi.dt_capacity(48 * 48, B) // 4
    ok, i, rr = rel_close(r["contrib"].cpu().numpy().ravel(), o["contrib"].ravel(), RTOL, ATOL)
    assert ok, (i, rr)
    r["ctx"].close()


def test_render_overflow_is_reported():
    """A context too small for the render's fan-out: the excess emits are
    dropped and counted, and the render reports RAFI_ERR_OVERFLOW."""
    dev = device()
    n, grid = 32, (2, 2, 2)
    vol = torch.from_numpy(W.blob_volume(n, 5)).to(dev)
    views = W.plusz_view(n, 32, 32)
    ctx = rafi.Context(8, rafi.DT_ITEM_BYTES, 32 * 32)          # room for the raygen only
    with pytest.raises(rafi.RafiError) as e:
        rafi.dt_render(vol, grid, views, 0.05, 1.0, 0.8, (0.0, 0.0, -1.0), 1.0, 2, 1, ctx=ctx)
    assert e.value.code == rafi.ERR_OVERFLOW
    assert ctx.stats()["dropped"] > 0
    ctx.close()
