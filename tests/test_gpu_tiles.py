"""The tile kernel's workgroup shapes and the binning's second set of bounds.

A launch of few tiles runs with fewer pixels per thread (1024, 512 or 256
threads per 32 x 32 tile); every shape has to give the bytes of the others.
The binning takes cameras whose pixels are not square through bounds of their
own, and its 4 x 4 groups of source blocks end unevenly.  Reference: the oracle, with the bars of the
parity tests (keys, holes and depth bit-exact, RGB within 1)."""
from dataclasses import replace

import numpy as np
import pytest

import scenegen as sg
from test_gpu_layered import compare_layered, run_layered
from test_gpu_learned import flat, rand_params
from test_gpu_parity import compare, ctx, fvv, gpu_run, say  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("path", ["plain", "layered", "learned"])
def test_workgroup_shapes_agree(fvv, ctx, oracle_lib, path):  # noqa: F811
    """77 tiles per view (ragged right and bottom): one view runs 1024
    threads a tile, 6 and 7 views lie on either side of 512 tiles, 13 and 14
    on either side of 1024."""
    import torch
    w = sg.config_small(60, n_cams=3, w=100, h=70, out_w=333, out_h=217, n_virtual=14, layered=path == "layered")
    views = w.virtual
    p = fvv.params(path={"plain": fvv.PATH_PLAIN, "layered": fvv.PATH_LAYERED, "learned": fvv.PATH_LEARNED}[path])
    ctx.set_rig(w.rig)
    if path == "layered":
        ctx.set_bg_model(w.bg_models)
    if path == "learned":
        ctx.net_load(flat(rand_params(61)))
    ctx.upload_mvd(w.frames)
    single = [ctx.synthesize(v, p=p) for v in views]
    for n in (6, 7, 13, 14):
        say(f"[gpu] {path}: {n} views of 333x217")
        outs = [torch.full((v.height, v.width, 3), 7, dtype=torch.uint8, device="cuda") for v in views[:n]]
        ctx.synthesize_batch(views[:n], outs, p=p)
        torch.cuda.synchronize()
        for a, o in zip(single, outs):
            assert np.array_equal(a, o.cpu().numpy())


def test_large_single_view_parity(fvv, ctx, oracle_lib):  # noqa: F811
    """One view on either side of each line: 27 x 19 (513), 32 x 32 (1024)
    and 33 x 32 tiles, the last row and column of one pixel."""
    w = sg.config_small(62, n_cams=3, w=160, h=100, out_w=834, out_h=577, n_virtual=1)
    for ow, oh in ((834, 577), (993, 993), (1025, 993)):
        v = w.virtual[0].with_size(ow, oh, 1.0)
        out, taps = gpu_run(fvv, ctx, w, v)
        compare(oracle_lib, w, v, out, taps)


@pytest.mark.parametrize("layered", [False, True])
@pytest.mark.parametrize("cw,ch,ratio", [(1, 1, 1.0), (33, 9, 1.4), (31, 65, 0.6), (96, 64, 3.0)])
def test_non_square_pixels_ragged_sources(fvv, ctx, oracle_lib, cw, ch, ratio, layered):  # noqa: F811
    """Sources whose 4 x 4 groups of blocks end unevenly (down to one pixel),
    with fy / fx = ratio."""
    w = sg.config_small(63, n_cams=3, w=cw, h=ch, out_w=150, out_h=90, n_virtual=2, layered=layered)
    w = replace(w, rig=[replace(c, fy=c.fy * ratio) for c in w.rig])
    v = replace(w.virtual[1], fy=w.virtual[1].fy * 1.2)
    if layered:
        out, taps = run_layered(fvv, ctx, w, v, max_fp=16.0)
        compare_layered(oracle_lib, w, v, out, taps, max_fp=16.0)
    else:
        out, taps = gpu_run(fvv, ctx, w, v, max_fp=16.0)
        compare(oracle_lib, w, v, out, taps, max_fp=16.0)


@pytest.mark.parametrize("fx", [1e7, 1e11, 1e20, 3e38])
def test_points_far_outside(fvv, ctx, oracle_lib, fx):  # noqa: F811
    """Focal lengths at which almost every point projects beyond the range of an
    int, of a float32 or to a NaN: none of them may leave a footprint."""
    w = sg.config_small(65, n_cams=3, w=96, h=64, out_w=150, out_h=90, n_virtual=2)
    for v in (replace(w.virtual[1], fx=fx, fy=fx), replace(w.virtual[1], fx=fx)):
        say(f"[gpu] virtual focal lengths {v.fx} {v.fy}")
        out, taps = gpu_run(fvv, ctx, w, v)
        compare(oracle_lib, w, v, out, taps)
