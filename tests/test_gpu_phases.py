"""Fixed pattern with B < 64: while the walks do not fill the chip four waves share
each row's and each key group's, else they are walked alone.  Walks shorter than the phases, of every remainder, empty
rows and columns, d = 32 / 64 / 128, with and without two-part products, and the
same bits on every run; against the fp64 oracle."""
import pytest
import torch

from oracle import oracle as orc_mod
from paper_1904_10509_amd import sparse_attn as sa
from paper_1904_10509_amd.inputs import make_inputs

from gpu_util import check_all, device, oracle_inputs, run_gpu

pytestmark = pytest.mark.gpu

F, P = sa.SA_FIXED, sa.SA_FIXED_PER_HEAD
A2, MG, IL = sa.SA_MODE_A2, sa.SA_MODE_MERGED, sa.SA_MODE_INTERLEAVED


# (pattern, mode, n, B, l, c, d, batch, heads)
@pytest.mark.parametrize("pattern,mode,n,B,l,c,d,batch,heads", [
    (F, MG, 32, 32, 32, 8, 64, 1, 1),       # one block
    (F, MG, 96, 32, 64, 16, 128, 1, 2),
    (F, MG, 352, 32, 96, 32, 64, 2, 1),     # walks of every remainder; blocks straddle l-blocks
    (F, A2, 416, 32, 128, 32, 128, 1, 2),   # empty rows and columns
    (F, IL, 672, 32, 128, 32, 64, 2, 3),
    (P, MG, 640, 32, 64, 16, 32, 1, 5),
    (F, MG, 16, 16, 16, 4, 32, 1, 1),
    (F, IL, 336, 16, 25, 25, 128, 1, 4),
    (F, A2, 304, 16, 48, 1, 64, 1, 3),      # two-part products
    (P, A2, 400, 16, 40, 10, 128, 2, 2),
    (F, MG, 1040, 16, 64, 2, 32, 1, 2),
])
def test_shared_walks(pattern, mode, n, B, l, c, d, batch, heads):
    run(pattern, mode, n, B, l, c, d, batch, heads)


# the other side of walk_phases: enough walks to fill the chip, each walked alone
@pytest.mark.parametrize("pattern,mode,n,B,l,c,d,batch,heads", [
    (F, MG, 512, 32, 128, 32, 64, 8, 16),
    (F, A2, 512, 32, 64, 1, 32, 2, 32),     # two-part products
    (F, IL, 512, 16, 64, 8, 128, 4, 8),     # the same at d = 128
    (P, MG, 512, 32, 64, 16, 128, 4, 8),
    (F, MG, 336, 16, 25, 25, 32, 8, 16),
    (F, MG, 512, 16, 1000, 32, 64, 4, 16),  # one l-block: long walks inside it alone
])
def test_walks_alone(pattern, mode, n, B, l, c, d, batch, heads):
    run(pattern, mode, n, B, l, c, d, batch, heads)


def run(pattern, mode, n, B, l, c, d, batch, heads):
    x = make_inputs(batch, heads, n, d, torch.bfloat16, seed=n + l + c + d)
    kw = dict(n=n, block=B, l=l, c=c, pattern=pattern, mode=mode, scale=d ** -0.5)
    got, again = run_gpu(x, **kw, dev=device()), run_gpu(x, **kw)
    assert all((got[name] == again[name]).all() for name in ("dq", "dk", "dv"))
    ref = orc_mod.backward(*oracle_inputs(x), pattern=pattern, mode=mode, l=l, c=c, scale=d ** -0.5)
    check_all(f"phases p{pattern} m{mode} n{n} B{B} l{l} c{c} d{d} {batch}x{heads}", got, ref, torch.bfloat16,
              names=("o", "lse", "dq", "dk", "dv"))
