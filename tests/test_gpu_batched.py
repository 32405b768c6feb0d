"""GPU batched form: many uneven scenes per launch.

Every scene's image must be bit-identical to rendering that scene alone with
the plain path (same per-ray arithmetic, different scheduling), for every
tuning (graph replay or direct launches, tile sizes, workgroup sizes), and
within 1e-5 of the float64 oracle."""
import numpy as np
import pytest
import torch

from gpu_util import announce, device, rel_close
from paper_2605_30294_amd import autotune, rafi
from paper_2605_30294_amd import workloads as W

pytestmark = pytest.mark.gpu

C32 = float(np.float32(0.025))
RTOL, ATOL = 1e-5, 1e-35


def _plain_images(vols, scenes):
    imgs, rounds = [], []
    for n, grid, view, off in scenes:
        v = vols[off:off + n ** 3].reshape(n, n, n)
        r = rafi.ea_render(v, grid, np.array([view]), c=C32)
        imgs.append(r["image"])
        rounds.append(r["rounds"])
        r["ctx"].close()
    return torch.cat(imgs), max(rounds)


def _small_batch(dev):
    specs = W.draw_scenes(12, seed=77, n_range=(8, 48), rays_side_range=(5, 40))
    views = []
    for i, sp in enumerate(specs):
        if i % 3 == 2:   # some scenes get a rotated view
            views.append(W.random_views(1, sp.n, sp.rays_side, sp.rays_side + 3, seed=300 + i)[0])
        else:
            views.append(W.plusz_view(sp.n, sp.rays_side, sp.rays_side)[0])
    vols, scenes = rafi.build_batch_inputs(specs, dev, views=views)
    return specs, vols, scenes


@pytest.mark.parametrize("tuning", [
    dict(),
    dict(use_graph=False, rounds_per_sync=1),
    dict(split_tile=1024, march_block=64, march_grid=7, rounds_per_sync=2),
    dict(split_tile=8192, march_block=512, march_grid=3000, use_graph=True, rounds_per_sync=16),
])
def test_batched_equals_plain_and_oracle(orc, tuning):
    dev = device()
    specs, vols, scenes = _small_batch(dev)
    announce(f"batched small {tuning}")
    b = rafi.Batch(scenes, c=C32)
    if tuning:
        b.set_tuning(**{**dict(split_tile=4096, march_block=256, march_grid=2048, use_graph=True,
                               rounds_per_sync=4), **tuning})
    image = torch.full((b.n_rays,), -7.0, dtype=torch.float32, device=dev)
    rounds = b.render(vols, image)
    plain, plain_rounds = _plain_images(vols, scenes)
    torch.cuda.synchronize()
    assert rounds == plain_rounds
    assert torch.equal(image, plain)
    img = image.cpu().numpy()
    vh = vols.cpu().numpy()
    base = 0
    for n, grid, view, off in scenes:
        m = int(view["width"]) * int(view["height"])
        o = orc.ea_render(vh[off:off + n ** 3].reshape(n, n, n), grid, np.array([view]), c=C32)
        ok, i, r = rel_close(img[base:base + m], o["image"], RTOL, ATOL)
        assert ok, (n, grid, i, r)
        base += m
    b.close()


def test_batched_repeat_and_graph_replay():
    """Several renders in a row through one captured graph give the same image."""
    dev = device()
    specs, vols, scenes = _small_batch(dev)
    b = rafi.Batch(scenes, c=C32)
    first = torch.empty(b.n_rays, dtype=torch.float32, device=dev)
    b.render(vols, first)
    for _ in range(3):
        again = torch.zeros_like(first)
        b.render(vols, again)
        torch.cuda.synchronize()
        assert torch.equal(first, again)
    b.close()


def test_batched_256_scenes(orc, tmp_path, monkeypatch):
    """256 uneven scenes (edges 32-256, 1-64 domains, 1K-1M rays): autotuned
    batched render equals the per-scene plain renders bit for bit; the oracle
    checks a seeded sample of rays of eight scenes."""
    dev = device()
    monkeypatch.setenv("RAFI_TUNE_CACHE", str(tmp_path / "tune.json"))
    specs = W.draw_scenes(256)
    announce("batched 256 scenes")
    vols, scenes = rafi.build_batch_inputs(specs, dev)
    b = rafi.Batch(scenes, c=C32)
    image = torch.empty(b.n_rays, dtype=torch.float32, device=dev)
    best, ms, _ = autotune.tune_batch(b, vols, image, space={"split_tile": [4096], "march_block": [256],
                                                              "march_grid": [2048, 4096], "use_graph": [1],
                                                              "rounds_per_sync": [8]}, reps=1)
    b.render(vols, image)
    plain, _ = _plain_images(vols, scenes)
    torch.cuda.synchronize()
    assert torch.equal(image, plain)
    img = image.cpu().numpy()
    rng = np.random.default_rng(11)
    for s in rng.choice(len(scenes), 8, replace=False):
        n, grid, view, off = scenes[s]
        m = int(view["width"]) * int(view["height"])
        base = int(b.scenes[s].ray_base)
        ids = np.sort(rng.choice(m, min(m, 2000), replace=False))
        vol = vols[off:off + n ** 3].reshape(n, n, n).cpu().numpy()
        o = orc.ea_brute(vol, grid, np.array([view]), c=C32, ray_ids=ids)
        ok, i, r = rel_close(img[base + ids], o["image"], RTOL, ATOL)
        assert ok, (s, i, r)
    b.close()


@pytest.mark.parametrize("n_scenes", [1, 63, 65, 4097])
def test_batched_scene_search(n_scenes):
    """Scene and domain counts around the steps of the 64-probe search, scenes
    smaller than a wavefront, rays that all miss: the plain renders' bits."""
    dev = device()
    specs, vols, scenes = _small_batch(dev)
    tiny = []
    for i, (n, grid, view, off) in enumerate(scenes):
        view = view.copy()
        view["width"], view["height"] = 1 + i % 5, 1 + i // 3   # 1 to 20 rays
        if i == 7:
            view["n_samples"] = 0
        tiny.append((n, grid, view, off))
    plain, plain_rounds = _plain_images(vols, tiny)
    sizes = [int(v["width"]) * int(v["height"]) for _, _, v, _ in tiny]
    whole, rest = divmod(n_scenes, len(tiny))
    want = torch.cat([plain] * whole + [plain[:sum(sizes[:rest])]])
    announce(f"batched scene search {n_scenes}")
    b = rafi.Batch([tiny[i % len(tiny)] for i in range(n_scenes)], c=C32)
    image = torch.full((b.n_rays,), -7.0, dtype=torch.float32, device=dev)
    for _ in range(2):
        rounds = b.render(vols, image)
        torch.cuda.synchronize()
        assert torch.equal(image, want)
        assert rounds == plain_rounds or n_scenes < len(tiny)
    b.close()


def test_batched_round_limit():
    """The limit counts the round that finds nothing left, as before: one round
    too few is refused, and the render after it is whole."""
    dev = device()
    _, vols, scenes = _small_batch(dev)
    b = rafi.Batch(scenes, c=C32)
    image = torch.empty(b.n_rays, dtype=torch.float32, device=dev)
    rounds = b.render(vols, image)
    want = image.clone()
    with pytest.raises(Exception):
        b.render(vols, image, max_rounds=rounds - 1)
    image.fill_(-7.0)
    b.render(vols, image, max_rounds=rounds)
    torch.cuda.synchronize()
    assert torch.equal(image, want)
    b.close()


def test_batched_graph_follows_its_workspace():
    """A tuning that grows the count table and is then put back: the round
    captured before held the table that the change freed. The render after it
    is the first one's, and allocations made in between keep their contents."""
    dev = device()
    _, vols, scenes = _small_batch(dev)
    announce("batched graph and workspace")
    b = rafi.Batch(scenes, c=C32)
    image = torch.empty(b.n_rays, dtype=torch.float32, device=dev)
    b.render(vols, image)
    want = image.clone()
    base = dict(split_tile=4096, march_block=256, march_grid=32768, use_graph=True, rounds_per_sync=4)
    for tile in (1024, 2048):
        b.set_tuning(**{**base, "split_tile": tile})
        held = [torch.full((1 << k,), 7, dtype=torch.int32, device=dev) for k in range(4, 14)]
        b.set_tuning(**base)
        image.fill_(-7.0)
        b.render(vols, image)
        torch.cuda.synchronize()
        assert torch.equal(image, want)
        assert all(bool((t == 7).all()) for t in held)
    b.close()


@pytest.mark.parametrize("kind", ["along z", "tilted", "thumbnails"])
def test_batched_march_kernels(kind):
    """Two large scenes and thirty of 5 x 5 to 6 x 6 rays over 64 bricks, whose
    wavefronts hold the slots of up to a dozen domains: along z the wavefronts of
    one or two domains and the listed others, tilted or without the large scenes
    every lane in its own domain. The plain renders' bits, twice (graph replay),
    and with the fewest workgroups."""
    dev = device()
    rng = np.random.default_rng(8)
    sizes = ([] if kind == "thumbnails" else [(32, (1, 2, 1), 311), (24, (2, 1, 3), 290)]) + \
        [(16, (4, 4, 4), 5 + i % 2) for i in range(30)]
    vols, scenes, off = [], [], 0
    for i, (n, grid, w) in enumerate(sizes):
        vols.append(torch.from_numpy(rng.random(n ** 3).astype(np.float32)).to(dev))
        tilt = i % 3 == 1 if kind == "along z" and i > 1 else kind != "along z"
        view = W.random_views(1, n, w, w, seed=70 + i)[0] if tilt else W.plusz_view(n, w, w)[0]
        scenes.append((n, grid, view, off))
        off += n ** 3
    vols = torch.cat(vols)
    announce(f"batched march {kind}")
    want, want_rounds = _plain_images(vols, scenes)
    b = rafi.Batch(scenes, c=C32)
    image = torch.full((b.n_rays,), -7.0, dtype=torch.float32, device=dev)
    for k in range(3):
        if k == 2:
            b.set_tuning(march_block=64, march_grid=1)
        image.fill_(-7.0)
        assert b.render(vols, image) == want_rounds
        torch.cuda.synchronize()
        assert torch.equal(image, want)
    b.close()
