"""NVFP4 calls that compute their own tensor absmax in the workspace: as
partial maxima (matrices up to 16 MB) or with one cleared value (larger)."""
import pytest
import torch

from paper_2608_13966_amd import quasar as Q
from paper_2608_13966_amd import synth

pytestmark = pytest.mark.gpu

# a stretch of one chunk; one and two workgroups; all 64 with a remainder; the
# last size that takes partial maxima and the first that does not
SHAPES = [(1, 16), (1, 8192), (1, 8208), (33, 16384), (513, 1040), (4096, 2048), (4097, 2048)]


@pytest.mark.parametrize("rows,cols", SHAPES)
@pytest.mark.parametrize("w_bf16", [True, False])
@pytest.mark.parametrize("where", ["first", "last", "middle"])
def test_workspace_absmax_matches_supplied(rows, cols, w_bf16, where):
    if not w_bf16 and rows * cols > 1 << 22:
        cols //= 2  # the same edge in bytes
    W, v, _ = synth.gen_matrix(rows, cols, 9, w_bf16=w_bf16, ema=False, device="cuda")
    n = W.numel()
    W.view(-1)[{"first": 0, "last": n - 1, "middle": n // 2 + 1}[where]] = -3.0  # the only |w| of its size
    amax = torch.zeros(4, device="cuda")
    amax[0] = 3.0
    assert float(W.float().abs().max()) == 3.0
    kw = dict(fmt="nvfp4", clips=(1.0, 0.9, 0.8))
    a = Q.reconstruct(W, v, None, **kw)
    a["workspace"].fill_(0xFF)  # a NaN in every slot: nothing of it may be read
    a = Q.reconstruct(W, v, None, out=a, **kw)
    b = Q.reconstruct(W, v, None, tensor_amax=amax, **kw)
    torch.cuda.synchronize()
    assert float(a["tensor_scale"][0]) == float(b["tensor_scale"][0])
    for k in ("codes", "scales", "r", "best_clip", "err"):
        assert torch.equal(a[k], b[k]), k


@pytest.mark.parametrize("rows,cols", SHAPES)
@pytest.mark.parametrize("g_fp32", [False, True])
def test_workspace_absmax_with_the_ema(rows, cols, g_fp32):
    """After the fused EMA the same load reads the partial maxima or the one value."""
    W, v, g = synth.gen_matrix(rows, cols, 11, w_bf16=True, ema=True, device="cuda")
    g = g.float() if g_fp32 else g
    amax = torch.zeros(4, device="cuda")
    amax[0] = W.abs().max()
    kw = dict(fmt="nvfp4", clips=(1.0, 0.9, 0.8))
    va, vb = v.clone(), v.clone()
    a = Q.reconstruct(W, v.clone(), g, **kw)
    a["workspace"].fill_(0xFF)
    a = Q.reconstruct(W, va, g, out=a, **kw)
    b = Q.reconstruct(W, vb, g, tensor_amax=amax, **kw)
    torch.cuda.synchronize()
    assert torch.equal(va, vb) and float(a["tensor_scale"][0]) == float(b["tensor_scale"][0])
    for k in ("codes", "scales", "r", "best_clip", "err"):
        assert torch.equal(a[k], b[k]), k


@pytest.mark.parametrize("rows", [8192, 8193])  # 256 MiB of bf16 W, the last with cached loads, and the next
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_absmax_around_the_last_level_cache(rows, dtype):
    cols = 16384 if dtype == torch.bfloat16 else 8192
    W = torch.zeros(rows, cols, dtype=dtype, device="cuda")
    a = torch.full((4,), 7.0, device="cuda")
    for at in (0, W.numel() // 2 + 1, W.numel() - 1):
        W.view(-1)[at] = -3.0
        s = Q.quasar_absmax(Q.Descriptor(rows, cols, fmt="nvfp4", bits=4, group=16, clips=(1.0,),
                                         w_dtype=Q.BF16 if dtype == torch.bfloat16 else Q.F32),
                            W, a, torch.cuda.current_stream().cuda_stream)
        assert s == Q.OK
        assert float(a[0]) == 3.0
        W.view(-1)[at] = 0.0
