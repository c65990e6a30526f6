"""C-ABI contract of libquasar.so, checked without a GPU: the library loads,
exports every entry point declared in include/quasar.h, and validates its
arguments on the host (quasar_check never touches device memory, so fake
aligned addresses stand in for device pointers here)."""
import os
import re

import numpy as np
import pytest

from paper_2608_13966_amd import quasar as Q

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
A = 0x10000  # a 16-byte aligned stand-in address (never dereferenced by quasar_check)


def declared_functions():
    src = open(os.path.join(ROOT, "include", "quasar.h")).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(quasar_[a-z_]+)\s*\(", src)))


def test_library_exports_every_declared_function():
    lib = Q.lib()
    names = declared_functions()
    assert set(names) == set(Q.EXPORTS), names
    for n in names:
        assert hasattr(lib, n), n
    assert Q.quasar_version().count(".") == 2


def test_status_strings():
    for s in (Q.OK, Q.ERR_ARG, Q.ERR_SHAPE, Q.ERR_ALIGN, Q.ERR_FORMAT, Q.ERR_WORKSPACE, Q.ERR_DEVICE):
        assert Q.quasar_status_string(s) and "unknown" not in Q.quasar_status_string(s)
    assert "unknown" in Q.quasar_status_string(42)


def _int_desc(**kw):
    args = dict(rows=64, cols=256, fmt="int", bits=4, group=128, clips=(1.0, 0.9, 0.8), w_dtype=Q.BF16)
    args.update(kw)
    rows, cols = args.pop("rows"), args.pop("cols")
    return Q.Descriptor(rows, cols, **args)


def _check(d, **ptrs):
    p = dict(W=A, v=A, g=None, codes=A, scales=A, zeros=A, r=A, best_clip=A, err=A, tensor_scale=None,
             tensor_amax=None, workspace=None, workspace_bytes=0)
    if d.desc.format == Q.NVFP4:
        p.update(zeros=None, tensor_scale=A)
    p.update(ptrs)
    return Q.quasar_check(d, p["W"], p["v"], p["g"], p["codes"], p["scales"], p["zeros"], p["r"], p["best_clip"],
                          p["err"], p["tensor_scale"], p["tensor_amax"], p["workspace"], p["workspace_bytes"])


def test_valid_int_and_nvfp4_descriptors():
    assert _check(_int_desc()) == Q.OK
    assert _check(_int_desc(bits=2, group=64, clips=tuple(np.linspace(1, 0.5, 12)))) == Q.OK
    d = _int_desc(fmt="nvfp4")
    assert _check(d, workspace=A, workspace_bytes=256) == Q.OK
    assert _check(d, tensor_amax=A) == Q.OK
    # optional outputs may be NULL
    assert _check(_int_desc(), r=None, best_clip=None, err=None) == Q.OK
    # variants: saliency weighting and deployed parameter precision
    for wt in ("h", "h2", "none"):
        for pd in ("fp32", "fp16", "bf16"):
            assert _check(_int_desc(weighting=wt, param_dtype=pd)) == Q.OK
        assert _check(_int_desc(fmt="nvfp4", weighting=wt), tensor_amax=A) == Q.OK


@pytest.mark.parametrize("kw,status", [
    (dict(bits=1), Q.ERR_FORMAT), (dict(bits=5), Q.ERR_FORMAT), (dict(group=32), Q.ERR_FORMAT),
    (dict(group=100), Q.ERR_FORMAT), (dict(cols=200), Q.ERR_SHAPE), (dict(rows=0), Q.ERR_SHAPE),
    (dict(cols=0), Q.ERR_SHAPE), (dict(rows=1 << 30, cols=1 << 20), Q.ERR_SHAPE),
    (dict(clips=()), Q.ERR_ARG), (dict(clips=tuple([1.0] * 17)), Q.ERR_ARG), (dict(clips=(1.0, 0.0)), Q.ERR_ARG),
    (dict(clips=(1.5,)), Q.ERR_ARG), (dict(clips=(-0.5,)), Q.ERR_ARG), (dict(clips=(float("nan"),)), Q.ERR_ARG),
    (dict(clips=(1e-9,)), Q.ERR_ARG), (dict(w_dtype=7), Q.ERR_FORMAT), (dict(w_dtype=Q.F16), Q.ERR_FORMAT),
    (dict(weighting=3), Q.ERR_ARG), (dict(weighting=-1), Q.ERR_ARG), (dict(param_dtype=5), Q.ERR_FORMAT),
    (dict(fmt="nvfp4", param_dtype="fp16"), Q.ERR_FORMAT),
])
def test_invalid_descriptors(kw, status):
    assert _check(_int_desc(**kw)) == status


def test_invalid_pointers_and_alignment():
    d = _int_desc()
    for name in ("W", "v", "codes", "scales", "zeros"):
        assert _check(d, **{name: None}) == Q.ERR_ARG, name
    for name in ("W", "v", "codes", "scales", "zeros", "r", "best_clip", "err"):
        assert _check(d, **{name: A + 8}) == Q.ERR_ALIGN, name
    assert _check(d, g=A, workspace_bytes=0) == Q.OK
    assert _check(d, g=A + 4) == Q.ERR_ALIGN
    # EMA decay range
    for b2 in (0.4, 1.0, float("nan")):
        assert _check(_int_desc(beta2=b2), g=A) == Q.ERR_ARG
    assert _check(_int_desc(beta2=0.5), g=A) == Q.OK
    assert _check(_int_desc(g_dtype=3), g=A) == Q.ERR_FORMAT
    assert _check(_int_desc(g_dtype=Q.F16), g=A) == Q.ERR_FORMAT
    nv = _int_desc(fmt="nvfp4")
    assert _check(nv, tensor_scale=None, workspace=A, workspace_bytes=256) == Q.ERR_ARG
    assert _check(nv) == Q.ERR_WORKSPACE
    assert _check(nv, workspace=A, workspace_bytes=255) == Q.ERR_WORKSPACE
    assert _check(_int_desc(fmt="nvfp4", group=16, cols=24)) == Q.ERR_SHAPE


def test_size_queries():
    d = _int_desc(rows=3, cols=384, bits=3, group=128)
    assert Q.quasar_num_groups(d) == 9
    assert Q.quasar_codes_bytes(d) == 9 * 48
    assert Q.quasar_workspace_bytes(d, False) == 0
    d = _int_desc(rows=5, cols=128, bits=2, group=64)
    assert Q.quasar_num_groups(d) == 10 and Q.quasar_codes_bytes(d) == 10 * 16
    d = _int_desc(rows=2, cols=64, fmt="nvfp4")
    assert Q.quasar_num_groups(d) == 8 and Q.quasar_codes_bytes(d) == 64
    assert Q.quasar_workspace_bytes(d, False) == 256 and Q.quasar_workspace_bytes(d, True) == 0
    assert Q.quasar_num_groups(_int_desc(cols=200)) == 0 and Q.quasar_codes_bytes(_int_desc(cols=200)) == 0


def test_absmax_entry_point_validation():
    """quasar_absmax rejects non-NVFP4 descriptors and bad pointers before
    launching anything."""
    d_int = _int_desc()
    assert Q.quasar_absmax(d_int, A, A, None) == Q.ERR_FORMAT
    nv = _int_desc(fmt="nvfp4")
    assert Q.quasar_absmax(nv, None, A, None) == Q.ERR_ARG
    assert Q.quasar_absmax(nv, A, None, None) == Q.ERR_ARG
    assert Q.quasar_absmax(nv, A + 4, A, None) == Q.ERR_ALIGN
    assert Q.quasar_absmax(_int_desc(fmt="nvfp4", cols=24), A, A, None) == Q.ERR_SHAPE


def _adam_check(d, opt=None, **ptrs):
    if opt is None:
        opt = Q.AdamW(1e-3, 0.9, 0.999, 1e-8, 0.01, 1)
    p = dict(W=A, m=A, v=A, g=A, codes=A, scales=A, zeros=A, r=A, r_dtype=Q.BF16, best_clip=A, err=A,
             tensor_scale=None, tensor_amax=None, amax_out=None)
    if d.desc.format == Q.NVFP4:
        p.update(zeros=None, tensor_scale=A, tensor_amax=A)
    p.update(ptrs)
    return Q.quasar_adamw_check(d, opt, p["W"], p["m"], p["v"], p["g"], p["codes"], p["scales"], p["zeros"],
                                p["r"], p["r_dtype"], p["best_clip"], p["err"], p["tensor_scale"],
                                p["tensor_amax"], p["amax_out"])


def test_adamw_entry_point_validation():
    f32 = _int_desc(w_dtype=Q.F32)
    assert _adam_check(f32) == Q.OK
    assert _adam_check(f32, r_dtype=Q.F32) == Q.OK
    assert _adam_check(_int_desc(beta2=0.0)) == Q.OK          # desc->beta2 is ignored
    assert _adam_check(_int_desc(), r_dtype=Q.F32) == Q.ERR_FORMAT   # bf16 W needs bf16 r
    assert _adam_check(f32, r_dtype=Q.F16) == Q.ERR_FORMAT
    nv = _int_desc(fmt="nvfp4", w_dtype=Q.F32)
    assert _adam_check(nv) == Q.OK
    assert _adam_check(nv, amax_out=A + 16) == Q.OK
    assert _adam_check(nv, amax_out=A) == Q.ERR_ARG            # the same buffer as tensor_amax
    assert _adam_check(nv, tensor_amax=None) == Q.ERR_ARG      # the tensor scale needs an amax
    assert _adam_check(f32, tensor_amax=A) == Q.ERR_ARG
    assert _adam_check(f32, amax_out=A) == Q.ERR_ARG
    assert _adam_check(nv, amax_out=A + 20) == Q.ERR_ALIGN
    for name in ("m", "g", "W", "v", "codes", "scales"):
        assert _adam_check(f32, **{name: None}) == Q.ERR_ARG, name
    assert _adam_check(f32, m=A + 8) == Q.ERR_ALIGN
    assert Q.quasar_adamw_check(f32, None, A, A, A, A, A, A, A, A, Q.BF16, A, A, None, None, None) == Q.ERR_ARG
    bad = [dict(step=0), dict(eps=0.0), dict(eps=float("inf")), dict(beta1=1.0), dict(beta1=-0.1),
           dict(beta2=0.4), dict(beta2=1.0), dict(lr=float("nan")), dict(lr=-1.0), dict(weight_decay=float("inf"))]
    for b in bad:
        hp = dict(lr=1e-3, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.01, step=1)
        hp.update(b)
        opt = Q.AdamW(hp["lr"], hp["beta1"], hp["beta2"], hp["eps"], hp["weight_decay"], hp["step"])
        assert _adam_check(f32, opt) == Q.ERR_ARG, b


def test_adamw_batch_validation():
    opt = Q.AdamW(1e-3, 0.9, 0.999, 1e-8, 0.01, 1)

    def mat(rows=64, cols=256, **kw):
        p = dict(W=A, m=A, v=A, g=A, codes=A, scales=A, zeros=A, r=A, best_clip=A, err=A, tensor_scale=None,
                 tensor_amax=None, amax_out=None)
        p.update(kw)
        return Q.AdamWMatrix(rows, cols, *[p[k] for k in ("W", "m", "v", "g", "codes", "scales", "zeros", "r",
                                                          "best_clip", "err", "tensor_scale", "tensor_amax",
                                                          "amax_out")])

    d = _int_desc(w_dtype=Q.F32)
    assert Q.quasar_adamw_batch_check(d, opt, [mat(), mat(rows=16, cols=128)], Q.BF16) == Q.OK
    assert Q.quasar_adamw_batch_check(d, opt, [], Q.BF16) == Q.ERR_ARG
    assert Q.quasar_adamw_batch_check(d, opt, [mat()] * (Q.MAX_BATCH + 1), Q.BF16) == Q.ERR_ARG
    assert Q.quasar_adamw_batch_check(d, None, [mat()], Q.BF16) == Q.ERR_ARG
    assert Q.quasar_adamw_batch_check(d, opt, [mat(), mat(m=None)], Q.BF16) == Q.ERR_ARG
    assert Q.quasar_adamw_batch_check(d, opt, [mat(), mat(cols=100)], Q.BF16) == Q.ERR_SHAPE
    assert Q.quasar_adamw_batch_check(_int_desc(), opt, [mat()], Q.F32) == Q.ERR_FORMAT  # bf16 W needs bf16 r
    nv = _int_desc(fmt="nvfp4", w_dtype=Q.F32)
    ok = dict(zeros=None, tensor_scale=A, tensor_amax=A)
    assert Q.quasar_adamw_batch_check(nv, opt, [mat(**ok), mat(**ok, amax_out=A + 16)], Q.BF16) == Q.OK
    assert Q.quasar_adamw_batch_check(nv, opt, [mat(**ok), mat(**dict(ok, tensor_amax=None))], Q.BF16) == Q.ERR_ARG
    # an amax_out is cleared before the pass: it may be no matrix's tensor_amax
    assert Q.quasar_adamw_batch_check(nv, opt, [mat(**dict(ok, tensor_amax=A + 32)),
                                                mat(**ok, amax_out=A + 32)], Q.BF16) == Q.ERR_ARG
    assert Q.quasar_adamw_batch_check(nv, opt, [mat(**ok, amax_out=A + 16), mat(**ok, amax_out=A + 16)],
                                      Q.BF16) == Q.ERR_ARG               # two matrices, one by-product buffer
    assert Q.quasar_adamw_batch_check(_int_desc(fmt="rubin", rows=16, cols=128), opt,
                                      [mat(16, 128, zeros=None)], Q.BF16) == Q.ERR_FORMAT


def test_rubin_descriptor_validation_and_sizes():
    d = _int_desc(fmt="rubin", rows=16, cols=128)
    assert _check(d, zeros=None) == Q.OK
    assert Q.quasar_num_groups(d) == 4
    assert Q.quasar_codes_bytes(d) == 4 * 192
    assert Q.quasar_workspace_bytes(d, 0) == 0
    assert _check(_int_desc(fmt="rubin", rows=12, cols=128), zeros=None) == Q.ERR_SHAPE
    assert _check(_int_desc(fmt="rubin", rows=16, cols=96), zeros=None) == Q.ERR_SHAPE
    assert _check(_int_desc(fmt="rubin", rows=16, cols=128, param_dtype="fp16"), zeros=None) == Q.ERR_FORMAT
    assert _check(d, zeros=None, tensor_amax=A) == Q.ERR_ARG
    assert _check(d, zeros=None, scales=None) == Q.ERR_ARG
    bad = Q.Descriptor(16, 128, fmt="rubin")
    bad.desc.group = 128
    assert _check(bad, zeros=None) == Q.ERR_FORMAT
    bad.desc.group, bad.desc.bits = 512, 4
    assert _check(bad, zeros=None) == Q.ERR_FORMAT
    # not fused with the optimiser step
    assert _adam_check(_int_desc(fmt="rubin", rows=16, cols=128, w_dtype=Q.F32), zeros=None) == Q.ERR_FORMAT


def test_symmetric_int_descriptor_validation():
    d = _int_desc(fmt="int_sym", bits=4, group=128)
    assert _check(d) == Q.OK and _check(d, zeros=None) == Q.OK
    assert _check(_int_desc(fmt="int_sym", bits=2, group=64, param_dtype="bf16"), zeros=None) == Q.OK
    assert _check(_int_desc(fmt="int_sym", bits=5)) == Q.ERR_FORMAT
    assert _check(_int_desc(fmt="int_sym", group=32)) == Q.ERR_FORMAT
    assert _check(d, tensor_amax=A) == Q.ERR_ARG
    assert _check(_int_desc(), tensor_amax=A) == Q.ERR_ARG
    assert Q.quasar_codes_bytes(_int_desc(fmt="int_sym", rows=2, cols=256, bits=3)) == 2 * 256 * 3 // 8
    assert _adam_check(_int_desc(fmt="int_sym", w_dtype=Q.F32)) == Q.ERR_FORMAT


def _mat(rows=64, cols=256, **kw):
    m = dict(rows=rows, cols=cols, W=A, v=A, g=None, codes=A, scales=A, zeros=A, r=A, best_clip=None, err=None,
             tensor_scale=None, tensor_amax=None)
    m.update(kw)
    return Q.Matrix(*[m[k] for k, _ in Q.Matrix._fields_])


def test_batch_entry_point_validation():
    d = _int_desc()
    assert Q.quasar_batch_check(d, [_mat(), _mat(rows=8, cols=128), _mat(rows=3, cols=384)]) == Q.OK
    assert Q.quasar_batch_check(d, []) == Q.ERR_ARG
    assert Q.quasar_batch_check(d, [_mat()] * 17) == Q.ERR_ARG
    assert Q.quasar_batch_check(d, [_mat(), _mat(g=A)]) == Q.ERR_ARG          # mixed EMA modes
    assert Q.quasar_batch_check(d, [_mat(), _mat(cols=200)]) == Q.ERR_SHAPE
    assert Q.quasar_batch_check(d, [_mat(), _mat(W=A + 8)]) == Q.ERR_ALIGN
    assert Q.quasar_batch_check(d, [_mat(zeros=None)]) == Q.ERR_ARG
    nv = _int_desc(fmt="nvfp4")
    assert Q.quasar_batch_check(nv, [_mat(zeros=None, tensor_scale=A, tensor_amax=A)] * 3) == Q.OK
    assert Q.quasar_batch_check(nv, [_mat(zeros=None, tensor_scale=A)]) == Q.ERR_ARG  # amax required
    rb = _int_desc(fmt="rubin")
    assert Q.quasar_batch_check(rb, [_mat(zeros=None), _mat(rows=16, cols=64, zeros=None)]) == Q.OK
    assert Q.quasar_batch_check(rb, [_mat(rows=12, zeros=None)]) == Q.ERR_SHAPE


def test_absmax_batch_validation():
    nv = _int_desc(fmt="nvfp4")
    mats = [_mat(), _mat(rows=1, cols=16), _mat(rows=5, cols=48)]
    assert Q.quasar_absmax_batch_check(nv, mats, [A, A + 16, A + 32]) == Q.OK
    assert Q.quasar_absmax_batch_check(nv, [], []) == Q.ERR_ARG
    assert Q.quasar_absmax_batch_check(nv, [_mat()] * 17, [A] * 17) == Q.ERR_ARG
    assert Q.quasar_absmax_batch_check(nv, mats, [A, None, A]) == Q.ERR_ARG    # an output missing
    assert Q.quasar_absmax_batch_check(nv, mats, [A, A + 16, A + 36]) == Q.ERR_ALIGN
    assert Q.quasar_absmax_batch_check(nv, [_mat(W=A + 8)], [A]) == Q.ERR_ALIGN
    assert Q.quasar_absmax_batch_check(nv, [_mat(W=None)], [A]) == Q.ERR_ARG
    assert Q.quasar_absmax_batch_check(nv, [_mat(cols=24)], [A]) == Q.ERR_SHAPE  # not whole 16-blocks
    assert Q.quasar_absmax_batch_check(nv, [_mat(rows=0)], [A]) == Q.ERR_SHAPE
    assert Q.quasar_absmax_batch_check(_int_desc(), [_mat()], [A]) == Q.ERR_FORMAT
    # one output buffer for two matrices would hold the larger of both maxima
    assert Q.quasar_absmax_batch_check(nv, mats, [A, A + 16, A]) == Q.ERR_ARG
    assert Q.quasar_absmax_batch_check(nv, mats, [A, A + 16, A + 32]) == Q.OK


def test_status_values():
    """The numeric status codes, as include/quasar.h declares them (QUASAR_OK
    0, then ERR_ARG -1, ERR_SHAPE -2, ERR_ALIGN -3, ERR_FORMAT -4,
    ERR_WORKSPACE -5, ERR_DEVICE -6), read from the header itself and from the
    library's status strings."""
    src = open(os.path.join(ROOT, "include", "quasar.h")).read()
    body = re.search(r"typedef enum \{(.*?)\} quasar_status;", src, flags=re.S).group(1)
    body = re.sub(r"/\*.*?\*/", "", body, flags=re.S)
    declared = {k: int(v) for k, v in re.findall(r"(QUASAR_[A-Z_]+)\s*=\s*(-?\d+)", body)}
    assert declared == {"QUASAR_OK": 0, "QUASAR_ERR_ARG": -1, "QUASAR_ERR_SHAPE": -2, "QUASAR_ERR_ALIGN": -3,
                        "QUASAR_ERR_FORMAT": -4, "QUASAR_ERR_WORKSPACE": -5, "QUASAR_ERR_DEVICE": -6}
    assert (Q.OK, Q.ERR_ARG, Q.ERR_SHAPE, Q.ERR_ALIGN, Q.ERR_FORMAT, Q.ERR_WORKSPACE, Q.ERR_DEVICE) == \
        (0, -1, -2, -3, -4, -5, -6)
    assert "workspace" in Q.quasar_status_string(-5) and "launch" in Q.quasar_status_string(-6)


def test_batch_wrappers_reject_mixed_matrices_before_launch():
    """The batched Python wrappers apply one descriptor to every matrix; a
    matrix whose dtype or shape differs from what that descriptor says is
    refused before anything is allocated or launched (CPU tensors here: the
    checks run first, so no device is touched)."""
    import torch
    W32 = torch.zeros(8, 128, dtype=torch.float32)
    W16 = torch.zeros(8, 128, dtype=torch.bfloat16)
    v = torch.zeros(8, 128, dtype=torch.float32)
    g = torch.zeros(8, 128, dtype=torch.bfloat16)
    with pytest.raises(ValueError, match="dtype"):
        Q.reconstruct_batch([(W32, v, None), (W16, v, None)], fmt="int", bits=4, group=128)
    with pytest.raises(ValueError, match="gradient"):
        Q.reconstruct_batch([(W16, v, g), (W16, v, None)], fmt="int", bits=4, group=128)
    with pytest.raises(ValueError, match="g must"):
        Q.reconstruct_batch([(W16, v, g), (W16, v, g.float())], fmt="int", bits=4, group=128)
    with pytest.raises(ValueError, match="v must"):
        Q.reconstruct_batch([(W16, v, g), (W16, v[:4], g)], fmt="int", bits=4, group=128)
    with pytest.raises(ValueError, match="contiguous"):
        Q.reconstruct_batch([(W16, v, g), (W16.t().contiguous().t(), v, g)], fmt="int", bits=4, group=128)
    with pytest.raises(ValueError, match="tensor_amax"):
        Q.reconstruct_batch([(W16, v, None, torch.zeros(4, dtype=torch.float64))], fmt="nvfp4")
    m = torch.zeros_like(v)
    with pytest.raises(ValueError, match="dtype"):
        Q.adamw_reconstruct_batch([(W32, m, v, g), (W16, m, v, g)], lr=1e-3, fmt="int", bits=4, group=128)
    with pytest.raises(ValueError, match="m must"):
        Q.adamw_reconstruct_batch([(W32, m, v, g), (W32, m.double(), v, g)], lr=1e-3, fmt="int", bits=4,
                                  group=128)
    with pytest.raises(ValueError, match="g must"):
        Q.adamw_reconstruct_batch([(W32, m, v, g), (W32, m, v, g.float())], lr=1e-3, fmt="int", bits=4,
                                  group=128)
    with pytest.raises(ValueError, match="dtype"):
        Q.absmax_batch([W16, W32])


def _with_path(value, fn):
    old = os.environ.get("QUASAR_INT_PATH")
    if value is None:
        os.environ.pop("QUASAR_INT_PATH", None)
    else:
        os.environ["QUASAR_INT_PATH"] = value
    try:
        return fn()
    finally:
        if old is None:
            os.environ.pop("QUASAR_INT_PATH", None)
        else:
            os.environ["QUASAR_INT_PATH"] = old


def test_rubin_cell_search_choice():
    """How the Rubin kernel finds a weight's cell (host-only): the bucket table
    for the paper's 15-factor grid and other spread grids, the tree search for
    a grid too dense for three compares per bucket or with
    QUASAR_RUBIN_PATH=tree."""
    paper = tuple(np.float32(x) for x in np.round(np.arange(1.0, 0.29, -0.05), 2))
    spread = [paper, (1.0,), tuple(np.linspace(1.0, 0.3, 8).astype(np.float32)),
              tuple(np.linspace(1.0, 0.3, 16).astype(np.float32))]
    dense = tuple(np.linspace(1.0, 0.9, 16).astype(np.float32))
    for clips in spread:
        assert Q.quasar_int_path(_int_desc(fmt="rubin", clips=clips)) == 1, clips
    assert Q.quasar_int_path(_int_desc(fmt="rubin", clips=dense)) == 0
    old = os.environ.get("QUASAR_RUBIN_PATH")
    os.environ["QUASAR_RUBIN_PATH"] = "tree"
    try:
        assert Q.quasar_int_path(_int_desc(fmt="rubin", clips=paper)) == 0
    finally:
        if old is None:
            os.environ.pop("QUASAR_RUBIN_PATH", None)
        else:
            os.environ["QUASAR_RUBIN_PATH"] = old


def test_int_path_choice():
    """Which INT kernel serves a clip grid (host-only).  By default the binned
    kernel takes grids with few code thresholds per group lane (INT2, INT3 with
    8 clips) and the direct kernel the rest (INT4 with 8 clips: about 110
    thresholds); QUASAR_INT_PATH=binned takes the binned kernel wherever its
    tables fit, QUASAR_INT_PATH=direct never."""
    grid8 = tuple(np.linspace(1.0, 0.65, 8).astype(np.float32))
    grid12 = tuple(np.linspace(1.0, 0.5, 12).astype(np.float32))
    grid16 = tuple(np.linspace(1.0, 0.3, 16).astype(np.float32))
    default_binned = [dict(bits=2, group=64, clips=grid12), dict(bits=3, group=128, clips=grid8),
                      dict(bits=2, group=128, clips=grid16), dict(fmt="int_sym", bits=3, group=128, clips=grid8)]
    fit_only = [dict(bits=4, group=128, clips=grid8), dict(fmt="int_sym", bits=4, group=128, clips=grid8),
                dict(bits=3, group=64, clips=grid8)]
    never = [dict(bits=4, group=64, clips=grid8), dict(bits=4, group=128, clips=grid16)]
    for kw in default_binned:
        assert Q.quasar_int_path(_int_desc(**kw)) == 1, kw
    for kw in fit_only + never:
        assert Q.quasar_int_path(_int_desc(**kw)) == 0, kw
    for kw in default_binned + fit_only:
        assert _with_path("binned", lambda: Q.quasar_int_path(_int_desc(**kw))) == 1, kw
    for kw in never:
        assert _with_path("binned", lambda: Q.quasar_int_path(_int_desc(**kw))) == 0, kw
    for kw in default_binned:
        assert _with_path("direct", lambda: Q.quasar_int_path(_int_desc(**kw))) == 0, kw
    assert Q.quasar_int_path(_int_desc(fmt="nvfp4")) == Q.ERR_FORMAT
    assert Q.quasar_int_path(_int_desc(bits=5)) == Q.ERR_FORMAT
    assert Q.quasar_int_path(_int_desc(clips=(1.0, 1.5))) == Q.ERR_ARG


@pytest.mark.parametrize("fmt,bits,group,k,least", [
    ("int", 3, 64, 9, 5 << 19), ("int", 3, 64, 10, 7 << 19), ("int_sym", 3, 64, 9, 5 << 19),
    ("int_sym", 3, 64, 10, 6 << 20), ("int_sym", 4, 128, 9, 6 << 20), ("int_sym", 3, 128, 14, 1 << 19),
    ("int_sym", 3, 128, 16, 1 << 19), ("int", 3, 128, 13, 0), ("int", 3, 128, 16, 0), ("int", 2, 64, 16, 0)])
def test_int_path_by_size(fmt, bits, group, k, least):
    """Grids for which the binned kernel is the faster one from some size on."""
    kw = dict(fmt=fmt, bits=bits, group=group, clips=tuple(np.linspace(1.0, 0.5, k)), cols=1024)
    rows = least // 1024
    assert Q.quasar_int_path(_int_desc(rows=max(rows, 1), **kw)) == 1
    if rows:
        assert Q.quasar_int_path(_int_desc(rows=rows - 1, **kw)) == 0
        assert _with_path("binned", lambda: Q.quasar_int_path(_int_desc(rows=1, **kw))) == 1


class _ArrayLike:
    def __array__(self, dtype=None, copy=None):
        return np.array([1.0, 0.8], dtype=dtype or np.float64)


def _readonly():
    a = np.array([1.0, 0.9], dtype=np.float32)
    a.flags.writeable = False
    return a


@pytest.mark.parametrize("clips", [
    1.0, 1, np.float32(0.9), "0.9", b"12", [[1.0, 0.9], [0.8, 0.7]], ["1.0", "0.9"], (1, 0.9), [], [None], None,
    _ArrayLike(), _readonly(), np.array(0.9), np.array([[1.0, 0.9]]), np.linspace(1, 0.5, 8)[::2],
    np.array([1.0, 0.5], dtype=object), np.zeros(0, dtype=np.float32), tuple(np.linspace(1, 0.3, 20))],
    ids=lambda c: type(c).__name__)
def test_clips_take_what_numpy_takes(clips):
    """Any form numpy makes a float32 array of gives that array's values, in its order."""
    want = np.ascontiguousarray(np.asarray(clips, dtype=np.float32))
    d = Q.Descriptor(64, 256, clips=clips)
    assert d.desc.n_clips == want.size
    np.testing.assert_array_equal([d.desc.clip_ratios[i] for i in range(want.size)], want.ravel())
    assert d.clips.dtype == np.float32 and d.clips.shape == want.shape
    np.testing.assert_array_equal(d.clips, want)


@pytest.mark.parametrize("clips", [{1.0, 0.9}, {1.0: 1}, (f for f in (1.0,)), [1j]], ids=lambda c: type(c).__name__)
def test_clips_refuse_what_numpy_refuses(clips):
    with pytest.raises(TypeError):
        Q.Descriptor(64, 256, clips=clips)


def test_clips_are_the_callers_array():
    """A contiguous float32 array is pointed to: an edit of it (or of d.clips)
    is an edit of the descriptor; d.clips may be assigned and changes nothing."""
    a = np.array([1.0, 0.9], dtype=np.float32)
    d = Q.Descriptor(64, 256, clips=a)
    a[1] = 0.5
    assert d.desc.clip_ratios[1] == 0.5 and d.clips is a
    d = Q.Descriptor(64, 256, clips=(1.0, 0.9))
    d.clips[1] = 0.25
    assert d.desc.clip_ratios[1] == 0.25
    d.clips = np.ones(2, dtype=np.float32)
    assert d.desc.clip_ratios[1] == 0.25


def test_tensors_off_the_gpu_are_refused_as_torch_does():
    """The current stream of a CPU tensor: torch's own error, type and text."""
    import torch
    W = torch.zeros(64, 256)
    with pytest.raises(Exception) as want:
        torch.cuda.current_stream(W.device)
    with pytest.raises(want.type) as got:
        Q.reconstruct(W, torch.zeros_like(W))
    assert str(got.value) == str(want.value)
