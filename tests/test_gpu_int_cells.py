"""The forms of the binned INT kernel against the oracle at the edges of their
tables: few and many cells (both sums of a cell at once, or one after the
other), grids whose thresholds need one, two or three compares per weight,
both group sizes and ragged row counts."""
import numpy as np
import pytest
import torch

from paper_2608_13966_amd import quasar as Q
from paper_2608_13966_amd import synth
from tests.test_gpu_parity import int_path, run_case

pytestmark = pytest.mark.gpu

# (fmt, bits, group, clips): the cells a group has, and what is at its edge
GRIDS = [
    ("int", 2, 64, (1.0,)),                                # 4 cells, the fewest
    ("int_sym", 2, 128, tuple(synth.clip_grid(1.0, 0.9, 16))),  # no tie cells; dense: three compares
    ("int", 2, 64, tuple(synth.clip_grid(1.0, 0.3, 16))),  # 35 cells, 10 a lane
    ("int", 3, 64, tuple(synth.clip_grid(1.0, 0.65, 8))),  # 51 cells: one sum at a time, 14 a lane
    ("int", 3, 64, tuple(synth.clip_grid(1.0, 0.5, 9))),   # 56 cells: the last with 14 a lane; two compares
    ("int", 3, 64, tuple(synth.clip_grid(1.0, 0.6, 10))),  # 63 cells, 16 a lane: the most for g64
    ("int", 3, 128, tuple(synth.clip_grid(1.0, 0.6, 11))),  # 68 cells
    ("int", 3, 128, tuple(synth.clip_grid(1.0, 0.5, 13))),  # 80 cells: the last with both sums at once
    ("int", 3, 128, tuple(synth.clip_grid(1.0, 0.65, 13))),  # 81 cells: the first with one, 12 a lane
    ("int", 3, 128, tuple(synth.clip_grid(1.0, 0.6, 13))),  # 79 cells
    ("int", 3, 128, tuple(synth.PAPER_CLIPS)),             # 91 cells; ties between clips in exact arithmetic: three compares
    ("int", 3, 128, (1.0, 1.0, 0.5, 0.5, 0.25, 0.25, 0.75, 0.75, 0.375)),  # equal and doubled factors
    ("int", 3, 128, tuple(synth.clip_grid(1.0, 0.3, 16))),  # 99 cells, 14 a lane
    ("int", 4, 128, tuple(synth.clip_grid(1.0, 0.65, 8))),  # 114 cells, 16 a lane, 15 steps
    ("int_sym", 4, 128, tuple(synth.clip_grid(1.0, 0.65, 9))),  # 127 cells, the most for g128, 14 steps
]


@pytest.mark.parametrize("fmt,bits,group,clips", GRIDS)
@pytest.mark.parametrize("w_bf16,ema,rows", [(True, True, 5), (False, False, 1)])
def test_binned_forms(fmt, bits, group, clips, w_bf16, ema, rows):
    """Random groups, and groups of range [-1, 1] (u = w exactly) whose weights
    sit on the code thresholds of every clip and one and two floats to either
    side, where the cell decides the codes."""
    cols = 3 * group
    with int_path("binned"):
        d = Q.Descriptor(rows, cols, fmt=fmt, bits=bits, group=group, clips=clips)
        assert Q.quasar_int_path(d) == 1
    name = f"cells.{fmt}{bits}.g{group}.K{len(clips)}.{'bf16' if w_bf16 else 'f32'}"
    run_case(name, rows, cols, 77, fmt=fmt, bits=bits, group=group, clips=clips, w_bf16=w_bf16, ema=ema)
    qm = (1 << (bits - 1)) - 1 if fmt == "int_sym" else (1 << bits) - 1
    pts = [0.0]
    for f in np.asarray(clips, dtype=np.float32):
        for b in range(1, (2 * qm if fmt == "int_sym" else qm) + 1):
            t = (b - qm - 0.5) * f / qm if fmt == "int_sym" else (b - qm / 2 - 0.5) * 2 * f / qm
            x = lo = hi = np.float32(t)
            for _ in range(2):
                lo, hi = np.nextafter(lo, np.float32(-2)), np.nextafter(hi, np.float32(2))
                pts += [lo, hi]
            pts.append(x)
    pts = np.asarray(pts, dtype=np.float32)
    rng = np.random.default_rng(5)
    W = rng.choice(pts, size=(8, cols)).astype(np.float32)
    W[:, ::group], W[:, 1::group] = -1.0, 1.0
    Wt = torch.from_numpy(W).cuda()
    v = torch.from_numpy(np.exp(rng.standard_normal(W.shape) * 3).astype(np.float32)).cuda()
    run_case(name + ".thresholds", *W.shape, 0, fmt=fmt, bits=bits, group=group, clips=clips, w_bf16=False, W=Wt, v=v)


@pytest.mark.parametrize("fmt,bits,group,k", [("int", 2, 64, 12), ("int", 3, 128, 15), ("int", 4, 128, 8),
                                              ("int_sym", 4, 128, 8), ("int_sym", 4, 64, 12), ("int_sym", 4, 128, 16)])
@pytest.mark.parametrize("w_bf16", [True, False])
def test_exact_path_sees_updated_saliency(fmt, bits, group, k, w_bf16):
    """Groups whose moments cannot fix the fit are evaluated from saliencies
    that the kernel reads again after the fused EMA stored them.  The gradient
    puts nearly all of v' on one weight and v on another, so the saliencies
    before the update give another fit."""
    rows, cols = 5, 3 * group
    rng = np.random.default_rng(k + group)
    W = (rng.standard_normal((rows, cols)) * 0.02).astype(np.float32)
    v = rng.random((rows, cols)).astype(np.float32) / group
    g = np.zeros((rows, cols), dtype=np.float32)
    for i in range(rows * cols // group):
        seg = slice(i * group, (i + 1) * group)
        at = i * group + rng.integers(1, group)
        v.flat[at - 1] = 1.0
        v.flat[seg] *= np.float32(10.0 ** -(6 + i % 4))
        g.flat[at] = 32.0
    Wt = torch.from_numpy(W).cuda()
    run_case(f"exact.ema.{fmt}{bits}.g{group}.K{k}.{w_bf16}", rows, cols, 0, fmt=fmt, bits=bits, group=group,
             clips=tuple(synth.clip_grid(1.0, 0.6, k)), w_bf16=w_bf16, ema=True,
             W=Wt.bfloat16() if w_bf16 else Wt, v=torch.from_numpy(v).cuda(), g=torch.from_numpy(g).cuda().bfloat16(),
             near_limit=rows * cols // group)


@pytest.mark.parametrize("bits,group,k", [(2, 64, 8), (3, 64, 4), (3, 128, 8), (3, 128, 15), (4, 128, 8)])
@pytest.mark.parametrize("rest", [0.0, 1e-25])
def test_symmetric_groups_with_their_saliency_on_code_0(bits, group, k, rest):
    """sum h q^2 is 0, or a saliency far below the fixed point's last place:
    the scale is RTN's, or the one that saliency fixes.  The other saliencies
    span e^+-20, so that the cell sums fill more than the 53 bits of an fp64."""
    rows, cols = 64, 4 * group
    rng = np.random.default_rng(k + group)
    W = (rng.standard_normal((rows, cols)) * 1e-3).astype(np.float32)
    v = np.exp(rng.standard_normal((rows, cols)) * 6).astype(np.float32)
    W[:, ::group] = 0.37
    v[:, ::group] = rest * v.max()
    run_case(f"code0.int_sym{bits}.g{group}.K{k}.{rest}", rows, cols, 0, fmt="int_sym", bits=bits, group=group,
             clips=tuple(synth.clip_grid(1.0, 0.65, k)), w_bf16=False, W=torch.from_numpy(W).cuda(),
             v=torch.from_numpy(v).cuda())
