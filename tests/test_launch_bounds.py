"""Grids that the host code launches against the buffers that it allocated, and
the fitting routes it chooses, without a GPU: libdpse runs on a recording
stand-in for the HIP runtime (hip_recorder.c) in a process of its own."""
import ctypes
import dataclasses
import subprocess
import sys
from pathlib import Path

import pytest

HERE = Path(__file__).resolve().parent
ROOT = HERE.parent
MODES = {"fp64": 0, "bf16": 1, "fp16": 2, "mix_fp32": 3, "mix_fp16": 4, "fp64_tab": 5}


class Launch(ctypes.Structure):
    _fields_ = [("name", ctypes.c_char_p), ("grid", ctypes.c_uint32 * 3), ("block", ctypes.c_uint32 * 3),
                ("lds", ctypes.c_uint64), ("arg", ctypes.c_uint64 * 192)]


def _recorder(so):
    """The recorder and libdpse on top of it (call in a fresh process)."""
    rec = ctypes.CDLL(so, mode=ctypes.RTLD_GLOBAL)
    rec.rec_launch.restype = ctypes.POINTER(Launch)
    rec.rec_bytes.restype = ctypes.c_uint64
    rec.rec_bytes.argtypes = [ctypes.c_uint64]
    from paper_2410_22867_amd import dpse
    return rec, dpse.lib(), dpse


def _launches(rec):
    return [rec.rec_launch(k).contents for k in range(rec.rec_launches())]


def _check_counters(rec, natoms):
    """Every work-group of an embedding kernel has its column counter (a
    128-byte line): of a launch's buffers the one whose size is a multiple of
    lines per compute unit."""
    line = 128 * rec.rec_ncu()
    seen = 0
    for l in _launches(rec):
        name = l.name.decode()
        if "k_embed" not in name:
            continue
        sizes = [b for b in (rec.rec_bytes(a) for a in l.arg) if b and b % line == 0]
        assert len(sizes) == 1, (name, sizes)
        need = 128 * l.grid[0] * l.grid[1]
        assert need <= sizes[0], f"{name}: grid {list(l.grid)} needs {need} bytes of counters, {sizes[0]} allocated ({natoms} atoms)"
        seen += 1
    assert seen >= 2


def _counters(so, ntypes, w):
    rec, L, dpse = _recorder(so)
    import numpy as np
    from paper_2410_22867_amd import inputs as I
    sel = (46, 92, 24, 16)[:ntypes]
    desc = dataclasses.replace(I.WATER, ntypes=ntypes, sel=sel, emb=(w, 2 * w, 4 * w), fit=(32,) * 3, masses=(1.0,) * ntypes)
    c = dpse.make_desc(desc)
    p = np.zeros(desc.n_params)
    model, ctx = ctypes.c_void_p(), ctypes.c_void_p()
    assert L.dp_model_create(ctypes.byref(c), p.ctypes.data, p.size, ctypes.byref(model)) == 0
    assert L.dp_model_compress(model, 4.0, 8.0, 0.1) == 0
    box = np.diag([20.0] * 3).reshape(9)
    for n in (1, 3, 64, 700, 3072, 3073, 4100, 9001, 40000):
        for budget in (0, 1 << 40):
            assert L.dp_ctx_create(model, n, 1, budget, ctypes.byref(ctx)) == 0
            for mode in MODES.values():
                rec.rec_clear()
                d = [1 << 20] * 6  # device addresses the host never follows
                assert L.dp_compute(ctx, d[0], d[1], box.ctypes.data, n, d[2], mode, d[3], None, d[4], d[5], None) == 0
                if mode != MODES["fp64_tab"]:
                    assert L.dp_backward_params(ctx, d[0], d[1], None) == 0
                _check_counters(rec, n)
            assert L.dp_ctx_destroy(ctx) == 0


# width of the hidden layers, types, atoms, mode -> kernels of the fitting net that run
LAYER, PAIR, FIRST, DD, GEMM = "k_fit_layer_", "k_fit_pair_", "k_fit_first_", "k_fit_dd_f64", "k_fit_gemm_f64"
ROUTES = [
    # hidden layers one per launch only where that is the faster way
    (240, 2, 192, "fp64", {LAYER}, {PAIR}), (240, 2, 1280, "fp64", {LAYER}, {PAIR}), (240, 2, 1281, "fp64", {PAIR}, {LAYER}),
    (128, 2, 192, "fp64", {LAYER}, {PAIR}), (128, 2, 896, "fp64", {LAYER}, {PAIR}), (128, 2, 897, "fp64", {PAIR}, {LAYER}),
    (64, 2, 192, "fp64", {LAYER}, {PAIR}), (48, 2, 192, "fp64", {PAIR}, {LAYER}), (16, 2, 192, "fp64", {PAIR}, {LAYER}),
    (240, 2, 640, "bf16", {LAYER}, {PAIR}), (240, 2, 641, "bf16", {PAIR}, {LAYER}), (224, 2, 192, "bf16", {PAIR}, {LAYER}),
    (64, 2, 192, "fp16", {PAIR}, {LAYER}), (64, 1, 500, "bf16", {PAIR}, {LAYER}),
    (192, 2, 1024, "mix_fp32", {LAYER}, {PAIR}), (192, 2, 1025, "mix_fp32", {PAIR}, {LAYER}),
    (176, 2, 192, "mix_fp32", {PAIR}, {LAYER}), (64, 1, 864, "mix_fp16", {PAIR}, {LAYER}),
    # the first layer's backward product with its reduction shared by a work-group
    (192, 2, 1280, "fp64", {DD}, {GEMM}), (192, 2, 1281, "fp64", {GEMM}, {DD}), (176, 2, 768, "fp64", {GEMM}, {DD}),
    (16, 2, 1260, "fp64", {GEMM}, {DD}),
    # T, D and the first layer in one launch
    (240, 2, 1280, "mix_fp32", {FIRST}, set()), (240, 3, 853, "mix_fp32", {FIRST}, set()),
    (240, 3, 1260, "mix_fp32", set(), {FIRST}), (240, 3, 512, "bf16", {FIRST}, set()), (240, 3, 768, "bf16", set(), {FIRST}),
    (240, 3, 1770, "fp64", {FIRST}, set()),
]


def _routes(so):
    rec, L, dpse = _recorder(so)
    import numpy as np
    from paper_2410_22867_amd import inputs as I
    box = np.diag([20.0] * 3).reshape(9)
    rec.rec_set_ncu(256)
    for fw, ntypes, n, mode, some, none in ROUTES:
        desc = dataclasses.replace(I.WATER, ntypes=ntypes, sel=(46, 92, 24)[:ntypes], fit=(fw,) * 3, masses=(1.0,) * ntypes)
        c = dpse.make_desc(desc)
        p = np.zeros(desc.n_params)
        model, ctx = ctypes.c_void_p(), ctypes.c_void_p()
        assert L.dp_model_create(ctypes.byref(c), p.ctypes.data, p.size, ctypes.byref(model)) == 0
        assert L.dp_ctx_create(model, n, 1, 0, ctypes.byref(ctx)) == 0
        rec.rec_clear()
        d = [1 << 20] * 6
        assert L.dp_compute(ctx, d[0], d[1], box.ctypes.data, n, d[2], MODES[mode], d[3], None, d[4], d[5], None) == 0
        names = [l.name.decode() for l in _launches(rec)]
        for k in some:
            assert any(k in x for x in names), (fw, ntypes, n, mode, k)
        for k in none:
            assert not any(k in x for x in names), (fw, ntypes, n, mode, k)
        assert L.dp_ctx_destroy(ctx) == 0 and L.dp_model_destroy(model) == 0


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("rec") / "libhiprecorder.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-Wall", str(HERE / "hip_recorder.c"), "-o", so], check=True)
    return so


def _run(code):
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True,
                       env={**__import__("os").environ, "PYTHONPATH": f"{ROOT}:{HERE}"}, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]


@pytest.mark.parametrize("w", [25, 32])
@pytest.mark.parametrize("ntypes", [1, 2, 3, 4])
def test_column_counters_cover_every_embedding_grid(recorder, ntypes, w):
    _run(f"import test_launch_bounds as t; t._counters({recorder!r}, {ntypes}, {w})")


def test_fitting_routes(recorder):
    _run(f"import test_launch_bounds as t; t._routes({recorder!r})")
