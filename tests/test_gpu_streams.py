"""What a call leaves behind for other streams: a queue read on a second stream
right after the call that made it, and a context moved from one stream to
another between calls, hold what they hold after a full synchronisation. The
contents themselves are checked against the oracle elsewhere."""
import numpy as np
import pytest
import torch

from gpu_util import announce, device
from paper_2605_30294_amd import rafi
from paper_2605_30294_amd import workloads as W

pytestmark = pytest.mark.gpu

C32 = float(np.float32(0.025))


def _buffer(ctx):
    """Room for the context's queue, allocated and filled before the call under test."""
    b = torch.zeros((ctx.capacity, ctx.item_bytes), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    return b


def _read_at_once(ctx, side, now):
    """The queue as the side stream finds it now, and after everything is done."""
    n_in = ctx.view().n_in
    ctx.set_stream(side)
    rafi._check(rafi.lib().rafi_copy_queue(ctx.handle, rafi._dptr(now), None), "rafi_copy_queue")
    torch.cuda.synchronize()
    later, _ = ctx.copy_queue()
    ctx.set_stream()
    return now[:n_in], later


def test_queue_of_a_seed_on_another_stream():
    """16M particles: the seed's scatter takes hundreds of microseconds."""
    dev = device()
    n, D = 1 << 24, 64
    announce("streams: seed")
    g = torch.Generator(device=dev).manual_seed(5)
    p = torch.rand((n, 10), generator=g, device=dev)
    nb = rafi.NBody(p, D, virtual_capacity=D * D)
    side = torch.cuda.Stream()
    try:
        flipped = p.flip(0).contiguous()
        room = _buffer(nb.P)
        nb.reseed(flipped)
        now, later = _read_at_once(nb.P, side, room)
        assert later.shape[0] == n and torch.equal(now, later)
    finally:
        nb.close()


def test_queues_of_a_step_on_another_stream():
    dev = device()
    announce("streams: step")
    nb = rafi.NBody(rafi.nb_to_device(W.nbody_particles(20_000), dev), 32, theta=0.3)
    side = torch.cuda.Stream()
    try:
        rooms = [_buffer(nb.V), _buffer(nb.R)]
        for _ in range(3):
            nb.step(1e-3)
            for ctx, room in zip((nb.V, nb.R), rooms):
                now, later = _read_at_once(ctx, side, room)
                assert later.shape[0] > 0 and torch.equal(now, later)
    finally:
        nb.close()


def test_queue_of_a_refused_render_on_another_stream():
    """A round limit too small for the render: the queue of its last round."""
    dev = device()
    n, w, nv = 64, 512, 32
    vol = torch.from_numpy(W.blob_volume(n, 3)).to(dev)
    views = np.concatenate([W.plusz_view(n, w, w)] * nv)
    ctx = rafi.Context(8, rafi.EA_ITEM_BYTES, nv * w * w)
    side = torch.cuda.Stream()
    announce("streams: refused render")
    room = _buffer(ctx)
    for k in (1, 2, 1):
        with pytest.raises(rafi.RafiError) as e:
            rafi.ea_render(vol, (2, 2, 2), views, c=C32, ctx=ctx, max_rounds=k)
        assert e.value.code == rafi.ERR_MAX_ROUNDS
        now, later = _read_at_once(ctx, side, room)
        assert later.shape[0] == nv * w * w and torch.equal(now, later)
    ctx.close()


def test_renders_on_changing_streams():
    """One context, a new stream for every render, no synchronisation between."""
    dev = device()
    n, w = 64, 256
    vols = [torch.from_numpy(W.blob_volume(n, 11 + k)).to(dev) for k in range(2)]
    views = W.random_views(4, n, w, w, seed=12)
    n_rays = 4 * w * w
    want = [rafi.ea_render(v, (4, 2, 2), views, c=C32)["image"] for v in vols]
    ctx = rafi.Context(16, rafi.EA_ITEM_BYTES, n_rays)
    vdev = rafi.views_to_device(views, dev)
    images = [torch.zeros(n_rays, dtype=torch.float32, device=dev) for _ in range(8)]
    torch.cuda.synchronize()
    announce("streams: renders")
    streams = [torch.cuda.Stream() for _ in range(3)]
    for k, image in enumerate(images):
        ctx.set_stream(streams[k % 3])
        rafi.ea_render_job(ctx, rafi.ea_job(vols[k % 2], (4, 2, 2), vdev, 4, w, w, image, c=C32))
    torch.cuda.synchronize()
    for k, image in enumerate(images):
        assert torch.equal(image, want[k % 2]), k
    ctx.close()
