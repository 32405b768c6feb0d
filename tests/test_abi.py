"""The C ABI library loads and exports every symbol its headers declare;
argument validation rejects bad calls before touching a device (no GPU use)."""
import ctypes as C
import os
import re

import pytest

from paper_2605_30294_amd import rafi

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    names = set()
    for h in os.listdir(os.path.join(ROOT, "include")):
        if not h.endswith(".h"):
            continue
        text = open(os.path.join(ROOT, "include", h)).read()
        if "__device__" in text:     # device-side inline header: nothing to export
            continue
        for m in re.finditer(r"^(?:int|void|const char \*)\s*\*?\s*(rafi_\w+)\s*\(", text, re.M):
            names.add(m.group(1))
    return names


def test_library_exports_every_declared_symbol():
    L = rafi.lib()
    names = _declared()
    assert len(names) >= 20
    missing = [n for n in sorted(names) if not hasattr(L, n)]
    assert not missing, missing
    # and the binding declares a signature for each of them
    assert names <= set(rafi._SIGS), sorted(names - set(rafi._SIGS))


def test_argument_validation_without_device():
    L = rafi.lib()
    h = C.c_void_p()
    assert L.rafi_create(0, 16, 100, C.byref(h)) == rafi.ERR_ARG
    assert L.rafi_create(8, 6, 100, C.byref(h)) == rafi.ERR_ARG          # not a multiple of 4
    assert L.rafi_create(8, 512, 100, C.byref(h)) == rafi.ERR_ARG        # too large
    assert L.rafi_create(8, 16, 0, C.byref(h)) == rafi.ERR_ARG
    assert L.rafi_create(8, 16, 1 << 32, C.byref(h)) == rafi.ERR_ARG
    assert L.rafi_create(10000, 16, 100, C.byref(h)) == rafi.ERR_ARG     # too many domains
    b = C.c_uint64(0)
    assert L.rafi_multisplit_workspace(1 << 20, 0, 32, C.byref(b)) == rafi.ERR_ARG
    assert L.rafi_multisplit_workspace(1 << 20, 1024, 32, C.byref(b)) == rafi.RAFI_OK and b.value > 0
    # misaligned pointers are rejected before any launch
    assert L.rafi_multisplit(C.c_void_p(8), C.c_void_p(16), 10, 16, 4, C.c_void_p(32), C.c_void_p(64),
                             C.c_void_p(128), C.c_void_p(256), 1 << 20, None) == rafi.ERR_ARG
    for code in range(0, -9, -1):
        assert rafi.strerror(code) != "unknown error"
    assert L.rafi_round(None, None, None) == rafi.ERR_ARG
    assert L.rafi_ea_render(None, None, 1, None) == rafi.ERR_ARG
    assert L.rafi_sl_trace(None, None, None, 0, 1, None, None) == rafi.ERR_ARG
    assert L.rafi_open(None, 10, rafi.SLOTS_APPEND) == rafi.ERR_ARG
    assert L.rafi_dt_raygen(None, None) == rafi.ERR_ARG
    assert L.rafi_dt_trace(None, None) == rafi.ERR_ARG
    assert L.rafi_dt_render(None, None, 10, None) == rafi.ERR_ARG
    assert L.rafi_nb_workspace(1000, 0, C.byref(b)) == rafi.ERR_ARG
    assert L.rafi_nb_workspace(1000, 2048, C.byref(b)) == rafi.ERR_ARG
    assert L.rafi_nb_workspace(1000, 64, C.byref(b)) == rafi.RAFI_OK and b.value > 1000 * 40
    assert L.rafi_nb_splitters(None, 10, 4, None, None, None) == rafi.ERR_ARG
    assert L.rafi_nb_seed(None, None, None, 0) == rafi.ERR_ARG
    assert L.rafi_nb_step(None, None, None, None, None, None) == rafi.ERR_ARG
    # the no-allocation split refuses problems beyond its fixed scratch buffer
    # (checked before any device call) and misaligned pointers
    assert L.rafi_multisplit_noalloc(C.c_void_p(256), C.c_void_p(512), 1 << 26, 32, 4096, C.c_void_p(1024),
                                     C.c_void_p(2048), C.c_void_p(4096), None) == rafi.ERR_TOO_LARGE
    assert L.rafi_multisplit_noalloc(C.c_void_p(8), C.c_void_p(16), 10, 16, 4, C.c_void_p(32), C.c_void_p(64),
                                     C.c_void_p(128), None) == rafi.ERR_ARG
    assert L.rafi_split_set_variant(18) == rafi.ERR_ARG
    assert L.rafi_split_set_variant(-1) == rafi.ERR_ARG


@pytest.mark.parametrize("item_bytes", [4, 12, 32, 44, 48, 64, 20])
def test_split_workspace_serves_smaller_splits_and_other_shapes(item_bytes):
    """A workspace asked for once, for a caller's largest split, is enough for
    every smaller one (up to 4096 tiles of 1024 slots, where the tiles begin
    to grow) and under every scatter shape: its size is that of a table with a
    column of n_domains + 2 counts per tile of 1024 slots, the 512-byte head
    and the scan's partial sums, whatever plan the split takes. Sizes that the
    lockstep shape takes are left out from 2^21 slots on (it needs more)."""
    L = rafi.lib()
    b = C.c_uint64(0)

    def size(n, D):
        assert L.rafi_multisplit_workspace(n, D, item_bytes, C.byref(b)) == rafi.RAFI_OK
        return b.value

    def up(x):
        return -(-x // 256) * 256

    end = (1 << 21) - 1 if item_bytes in (12, 44, 20) else 4096 * 1024
    sizes = [1, 1024, 1025, 4096, 8192, 8193, 33_000, 126_976, 128_000, 258_049, 507_904, 507_905, 524_288, 525_312,
             1_000_000, 1_032_192, 1_036_288, 2_031_616, 2_032_640, 3_000_000, end]
    sizes = sorted({n for n in sizes if n <= end} | {1024 * k for k in range(1, end // 1024, 37)})
    try:
        for D in (1, 2, 5, 16, 64, 100, 128, 129, 200):
            got = []
            for n in sizes:
                tiles = -(-n // 1024)
                table = (D + 2) * tiles
                want = 512 + up(4 * table) + up(4 * -(-table // 4096))
                assert size(n, D) == want, (n, D)
                got.append(want)
            assert got == sorted(got)
        for variant in range(1, 17):
            rafi.split_set_variant(variant)
            for D in (2, 64, 128):
                for n in (8192, 126_976, 1_000_000, 2_031_616):
                    if n <= end:
                        other = size(n, D)
                        rafi.split_set_variant(0)
                        assert size(n, D) == other, (n, D, variant)
                        rafi.split_set_variant(variant)
    finally:
        rafi.split_set_variant(0)


def test_batch_tuning_defaults_are_the_librarys():
    """Batch.set_tuning fills in what a caller leaves out: a call that changes
    one field must not move the others from the library's defaults, which the
    header states."""
    import inspect
    text = open(os.path.join(ROOT, "include", "rafi.h")).read()
    struct = text[text.index("typedef struct rafi_batch_tuning {"):text.index("} rafi_batch_tuning;")]
    stated = {m.group(1): int(m.group(2)) for m in re.finditer(r"(\w+);\s*/\*[^*]*\(default (\d+)\)", struct)}
    given = {k: int(p.default) for k, p in inspect.signature(rafi.Batch.set_tuning).parameters.items() if k != "self"}
    assert len(stated) == 5 and given == stated


def test_dt_capacity_bound():
    """Capacity for delta tracking: 2 slots per visit x (the path + one shadow
    ray per scattering event) per path."""
    L = rafi.lib()
    cap = C.c_uint64(0)
    assert L.rafi_dt_capacity(1000, 4, C.byref(cap)) == rafi.RAFI_OK and cap.value == 2 * 1000 * 5
    assert L.rafi_dt_capacity(1000, 0, C.byref(cap)) == rafi.ERR_ARG
    assert L.rafi_dt_capacity(1 << 31, 1, C.byref(cap)) == rafi.ERR_ARG


def test_struct_layouts_match_header(tmp_path):
    """Every ctypes struct of the binding has the field offsets and size that a
    C compiler gives the header's struct (compiled here with gcc)."""
    import subprocess
    structs = {"rafi_device_view": rafi.DeviceView, "rafi_ea_job": rafi.EAJob, "rafi_sl_job": rafi.SLJob,
               "rafi_dt_job": rafi.DTJob, "rafi_nb_job": rafi.NBJob, "rafi_ortho_view": rafi.ViewRec, "rafi_ea_scene": rafi.SceneRec,
               "rafi_batch_tuning": rafi.BatchTuning, "rafi_stats_t": rafi.Stats, "rafi_profile": rafi.Profile}
    lines = ["#include <stdio.h>", "#include <stddef.h>", '#include "rafi.h"', "int main(void) {"]
    for cname, cls in structs.items():
        lines.append(f'printf("{cname} size %zu\\n", sizeof({cname}));')
        for fname, _ in cls._fields_:
            lines.append(f'printf("{cname} {fname} %zu\\n", offsetof({cname}, {fname}));')
    lines.append("return 0; }")
    src = tmp_path / "layout.c"
    src.write_text("\n".join(lines))
    exe = tmp_path / "layout"
    subprocess.run(["gcc", "-std=c11", "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe)], check=True)
    got = {}
    for line in subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.splitlines():
        cname, key, val = line.split()
        got[(cname, key)] = int(val)
    for cname, cls in structs.items():
        assert got[(cname, "size")] == C.sizeof(cls), cname
        for fname, _ in cls._fields_:
            assert got[(cname, fname)] == getattr(cls, fname).offset, (cname, fname)


def test_python_layer_names():
    """The Python layer's entry points: a context with round(), the
    differentiable render, the streamline trace and the stateless split."""
    assert callable(rafi.Context.round)
    assert rafi.render is rafi.ea_render_differentiable
    assert rafi.trace_streamlines is rafi.sl_trace
    assert callable(rafi.multisplit)
    assert issubclass(rafi.EARender, __import__("torch").autograd.Function)


def test_binding_rejects_bad_volume_and_field_shapes():
    """The job builders check shape and dtype before any pointer reaches the
    library: a non-cubic or non-float32 volume or field would make the
    kernels read n^3 voxels past the allocation."""
    import torch
    views = None
    img = torch.empty(4)
    for vol in (torch.zeros(4, 4, 2), torch.zeros(4, 4, 4, dtype=torch.float16), torch.zeros(4, 4),
                torch.zeros(4, 4, 4, dtype=torch.float64)):
        with pytest.raises(ValueError):
            rafi.ea_job(vol, (1, 1, 1), views, 1, 2, 2, img)
    ep, st = torch.empty(1, 3), torch.empty(1, dtype=torch.int32)
    for f in (torch.zeros(8, 8, 4, 3), torch.zeros(8, 8, 8, 2), torch.zeros(8, 8, 8, 3, dtype=torch.float16),
              torch.zeros(8, 8, 8)):
        with pytest.raises(ValueError):
            rafi.sl_job(f, (1, 1, 1), ep, st)
    for f in (torch.zeros(8, 8, 4, 3), torch.zeros(8, 8, 8, 3, dtype=torch.float64)):
        with pytest.raises(ValueError):
            rafi.sl_pack(f)
