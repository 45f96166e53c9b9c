"""The fp32 matrix-core kernels at the edges of their tiles: strips of 16 rows
or columns shared by eight waves, walks with fewer entries than waves, every
block size and head size, patterns whose runs straddle the 16-wide groups,
strided views.  Bar: 1e-5 plus half an ulp against the fp64 oracle."""
import pytest
import torch

from oracle import oracle as orc_mod
from paper_1904_10509_amd import sparse_attn as sa
from paper_1904_10509_amd.inputs import make_inputs

from gpu_util import check_all, device, oracle_inputs, run_gpu, to64

pytestmark = pytest.mark.gpu

S, F, P = sa.SA_STRIDED, sa.SA_FIXED, sa.SA_FIXED_PER_HEAD
A1, A2, MG, IL = sa.SA_MODE_A1, sa.SA_MODE_A2, sa.SA_MODE_MERGED, sa.SA_MODE_INTERLEAVED


# (pattern, mode, n, B, l, c, d, batch, heads)
@pytest.mark.parametrize("pattern,mode,n,B,l,c,d,batch,heads", [
    (S, MG, 16, 16, 4, 0, 32, 1, 1),      # one strip, one tile
    (S, MG, 64, 64, 64, 0, 128, 1, 1),
    (S, MG, 336, 16, 7, 0, 64, 1, 3),     # 21 entries over eight waves; every tile partial
    (S, A2, 480, 32, 50, 0, 128, 2, 1),
    (S, IL, 448, 64, 64, 0, 64, 1, 3),
    (S, A1, 256, 32, 300, 0, 32, 1, 2),   # the dense limit
    (F, MG, 960, 64, 96, 40, 64, 1, 2),   # blocks straddle l-blocks, windows straddle groups
    (F, A2, 512, 32, 128, 8, 128, 1, 2),  # empty rows, half a group of summary keys
    (F, IL, 624, 16, 52, 13, 32, 2, 3),
    (F, A1, 512, 64, 128, 32, 64, 1, 2),
    (P, MG, 768, 64, 128, 32, 64, 1, 5),
    (P, A2, 320, 32, 40, 10, 32, 1, 4),
])
def test_f32_tiles(pattern, mode, n, B, l, c, d, batch, heads):
    x = make_inputs(batch, heads, n, d, torch.float32, seed=n + l + c + d)
    got = run_gpu(x, n=n, block=B, l=l, c=c, pattern=pattern, mode=mode, scale=d ** -0.5)
    ref = orc_mod.backward(*oracle_inputs(x), pattern=pattern, mode=mode, l=l, c=c, scale=d ** -0.5)
    check_all(f"f32 p{pattern} m{mode} n{n} B{B} l{l} c{c} d{d} {batch}x{heads}", got, ref, torch.float32,
              names=("o", "lse", "dq", "dk", "dv"))


def test_f32_views_and_repeats():
    """[b, n, h, d] storage seen as [b, h, n, d], and the same bits on every run."""
    dev = device()
    n, l, c, B, d, h = 512, 64, 16, 32, 64, 3
    x = make_inputs(2, h, n, d, torch.float32, seed=31)
    lay = sa.build_layout(n, B, l, c, F, MG, device=dev)
    q, k, v, dout = (x[name].transpose(1, 2).contiguous().to(dev).transpose(1, 2) for name in ("q", "k", "v", "dout"))
    runs = []
    for _ in range(2):
        o, lse = sa.forward(q, k, v, lay)
        runs.append((o, lse) + tuple(sa.backward(q, k, v, o, dout, lse, lay)))
    assert all(torch.equal(a, b) for a, b in zip(*runs))
    ref = orc_mod.backward(*oracle_inputs(x), pattern=F, mode=MG, l=l, c=c, scale=d ** -0.5)
    names = ("o", "lse", "dq", "dk", "dv")
    check_all("f32 [b, n, h, d] views", {name: to64(t) for name, t in zip(names, runs[0])}, ref, torch.float32, names=names)


def test_f32_small_weights():
    """Weights far below a row's largest to the precision of fp32: every key has a
    coordinate of V of its own and an exact score 0, -8.25, -8.5, ..., so that each
    element of O is one weight.  Bar: two exponentials of 1 ulp (a wave's maximum and
    the row's), 1 for the reciprocal, a rounding each for the products and the sum:
    4.5 * 2^-23."""
    dev = device()
    n = d = 64
    score = -(8.0 + 0.25 * torch.arange(n, dtype=torch.float64))
    score[0] = 0.0
    q, k = torch.zeros(2, 1, 1, n, d)
    q[..., 0] = 1.0
    k[..., 0] = score.float()
    v = torch.eye(n).reshape(1, 1, n, d)
    lay = sa.build_layout(n, 16, n, 0, S, A1, device=dev)
    o, _ = sa.forward(q.to(dev), k.to(dev), v.to(dev), lay, 1.0)
    w = torch.tril(torch.exp(score).expand(n, n))
    ref = w / w.sum(1, keepdim=True)
    err = ((o[0, 0].cpu().double() - ref).abs() / ref.clamp_min(1e-300)).tril().max().item()
    print(f"f32 small weights: relative error {err:.2e}", flush=True)
    assert err <= 4.5 * 2.0 ** -23
