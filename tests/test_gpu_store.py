"""How whole lines are stored depends on W's type, the mode and whether what a
launch reads and writes fits the last-level cache: the same bytes in every
case, and none past a tensor's end."""
import pytest
import torch

from paper_2608_13966_amd import quasar as Q
from paper_2608_13966_amd import synth

pytestmark = pytest.mark.gpu

COLS = 384
PAD = 4096  # bytes after a tensor's end that must stay as they are
# (fmt, bits, group, W bf16, mode, bytes read and written per weight)
CASES = [
    ("int", 4, 128, True, "none", 8), ("int", 4, 128, False, "adamw", 16), ("int", 2, 64, True, "ema", 10),
    ("int", 3, 64, False, "ema", 14), ("int_sym", 4, 64, True, "ema", 10), ("int", 2, 128, True, "adamw", 14),
    ("nvfp4", 4, 16, False, "adamw", 16), ("nvfp4", 4, 16, True, "adamw", 14), ("rubin", 3, 512, True, "ema", 10),
]


def _padded(rows, cols, dtype, src=None):
    """A [rows, cols] tensor followed by PAD bytes of 0xA5, and those bytes."""
    n = rows * cols * torch.empty(0, dtype=dtype).element_size()
    raw = torch.full((n + PAD,), 0xA5, dtype=torch.uint8, device="cuda")
    t = raw[:n].view(dtype).view(rows, cols)
    if src is not None:
        t.copy_(src)
    return t, raw[n:]


def _call(mode, W, m, v, g, out, **kw):
    if mode == "adamw":
        Q.adamw_reconstruct(W, m, v, g, lr=1e-3, weight_decay=0.01, step=2, out=out, r_dtype="bf16", **kw)
    else:
        Q.reconstruct(W, v, g, out=out, **kw)


@pytest.mark.parametrize("fmt,bits,group,wb,mode,per", CASES)
@pytest.mark.parametrize("where", ["fits", "does not fit"])
def test_stores_of_large_launches(fmt, bits, group, wb, mode, per, where):
    """One call, of a few times 10^6 bytes or just above the cache's size, against
    calls on slices of its rows; the last wavefront of the whole is ragged."""
    cols = 448 if fmt == "rubin" else COLS
    limit = (4 << 20) if where == "fits" else (256 << 20)
    rows = limit // (cols * per) // 8 * 8 + (8 if fmt == "rubin" else 13)
    step = 320
    clips = (1.0, 0.85, 0.7)
    W0, v0, g = synth.gen_matrix(rows, cols, 3, w_bf16=wb, ema=mode != "none", device="cuda")
    m0 = torch.randn(rows, cols, device="cuda") * 1e-4 if mode == "adamw" else None
    rd = torch.bfloat16 if mode == "adamw" else W0.dtype
    kw = dict(fmt=fmt, bits=bits, group=group, clips=clips)
    if fmt == "nvfp4":
        kw["tensor_amax"] = torch.tensor([float(W0.abs().max()), 0, 0, 0], device="cuda")

    def outputs(W, r):
        d = Q.Descriptor(*W.shape, fmt=fmt, bits=bits, group=group, clips=clips, w_dtype=Q.BF16 if wb else Q.F32)
        return dict(Q.alloc_outputs(d, W, want_r=False, has_amax=fmt == "nvfp4"), r=r, amax_out=None)

    pads = []
    (W, p), (v, q), (r, s) = (_padded(rows, cols, W0.dtype, W0), _padded(rows, cols, torch.float32, v0),
                              _padded(rows, cols, rd))
    m, t = _padded(rows, cols, torch.float32, m0) if mode == "adamw" else (None, s)
    pads += [p, q, s, t]
    print(f"[case] {fmt}{bits} {mode} {where} {rows}x{cols}", flush=True)
    _call(mode, W, m, v, g, outputs(W, r), **kw)
    torch.cuda.synchronize()
    assert all(bool((x == 0xA5).all()) for x in pads)
    for a in range(0, rows, step):
        z = slice(a, min(rows, a + step))
        Ws, vs, ms = W0[z].clone(), v0[z].clone(), None if m0 is None else m0[z].clone()
        rs = torch.empty(Ws.shape, dtype=rd, device="cuda")
        _call(mode, Ws, ms, vs, None if g is None else g[z], outputs(Ws, rs), **kw)
        for name, whole, part in (("W", W, Ws), ("v", v, vs), ("m", m, ms), ("r", r, rs)):
            assert whole is None or torch.equal(whole[z], part), (name, a)


@pytest.mark.parametrize("fmt,bits,group,mode", [("int", 2, 64, "ema"), ("int", 3, 128, "ema"), ("int_sym", 4, 128, "ema"),
                                                 ("int", 4, 128, "adamw"), ("int", 2, 64, "adamw")])
@pytest.mark.parametrize("rows", [2741, 87381])  # x 384, 14 bytes a weight or more: fits the cache, does not
def test_exact_path_reads_what_was_stored(fmt, bits, group, mode, rows):
    """Groups whose moments cannot fix the fit read v' again after it was
    stored; the gradient puts nearly all of it on another weight than v has it on.
    One call against calls on slices of its rows (such small calls are checked
    against the oracle elsewhere)."""
    rng = torch.Generator(device="cuda").manual_seed(7)
    n = rows * COLS // group
    W0 = torch.randn(rows, COLS, device="cuda", generator=rng) * 0.02
    v0 = torch.rand(n, group, device="cuda", generator=rng) / group
    at = torch.randint(1, group, (n, 1), device="cuda", generator=rng)
    v0.scatter_(1, at - 1, 1.0)
    v0 = (v0 * 1e-7).view(rows, COLS)
    g = torch.zeros(n, group, device="cuda").scatter_(1, at, 32.0).view(rows, COLS).bfloat16()
    m0 = torch.zeros_like(W0) if mode == "adamw" else None
    clips = tuple(float(x) for x in synth.clip_grid(1.0, 0.6, 8))
    kw = dict(fmt=fmt, bits=bits, group=group, clips=clips)
    keys = ("codes", "scales", "zeros", "best_clip", "err")

    def call(z):
        W, v, m = W0[z].clone(), v0[z].clone(), None if m0 is None else m0[z].clone()
        d = Q.Descriptor(*W.shape, w_dtype=Q.F32, **kw)
        r = torch.empty(W.shape, dtype=torch.bfloat16 if mode == "adamw" else W.dtype, device="cuda")
        out = dict(Q.alloc_outputs(d, W, want_r=False), r=r, amax_out=None)
        _call(mode, W, m, v, g[z], out, **kw)
        return dict(out, v=v)

    print(f"[case] exact {fmt}{bits} g{group} {mode} {rows}x{COLS}", flush=True)
    whole = call(slice(0, rows))
    parts = [call(slice(a, min(rows, a + 256))) for a in range(0, rows, 256)]
    for k in (*keys, "r", "v"):
        assert torch.equal(whole[k].flatten(), torch.cat([p[k].flatten() for p in parts])), k
