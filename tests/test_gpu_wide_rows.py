"""Many query blocks, walked one or, where the walks are long too, two per workgroup
(see wide_rows): an odd number of query blocks, one l-block per pair and several,
each head mode, the strided band and the dense limit, against the fp64 oracle."""
import pytest
import torch

from oracle import oracle as orc_mod
from paper_1904_10509_amd import sparse_attn as sa
from paper_1904_10509_amd.inputs import make_inputs

from gpu_util import check_all, oracle_inputs, run_gpu

pytestmark = pytest.mark.gpu

S, F, P = sa.SA_STRIDED, sa.SA_FIXED, sa.SA_FIXED_PER_HEAD
A1, A2, MG, IL = sa.SA_MODE_A1, sa.SA_MODE_A2, sa.SA_MODE_MERGED, sa.SA_MODE_INTERLEAVED


# (pattern, mode, n, l, c, batch, heads); B = d = 64
@pytest.mark.parametrize("pattern,mode,n,l,c,batch,heads", [
    (F, MG, 2112, 128, 32, 8, 8),     # 33 query blocks: 17 x 64 workgroups
    (F, A2, 2112, 256, 32, 8, 8),
    (F, IL, 2112, 128, 40, 8, 8),
    (F, A1, 2048, 384, 32, 8, 8),
    (P, MG, 2112, 128, 32, 8, 8),
    (F, MG, 2112, 128, 96, 8, 8),     # 16 far steps a row on average, 17 x 64 workgroups
    (F, A2, 2112, 128, 128, 8, 8),
    (F, IL, 2112, 128, 96, 8, 8),
    (F, A1, 2112, 2048, 32, 16, 8),   # 17 x 128 workgroups, one long l-block and the start of another
    (P, MG, 4416, 128, 32, 6, 8),     # summary halves in pairs, 35 x 48 workgroups
    (S, A1, 2112, 500, 0, 8, 8),      # a band of eight blocks and the diagonal one
    (S, MG, 2112, 5000, 0, 8, 8),     # the dense limit
])
def test_pairs_of_query_blocks(pattern, mode, n, l, c, batch, heads):
    d = 64
    x = make_inputs(batch, heads, n, d, torch.bfloat16, seed=n + l + c + mode)
    got = run_gpu(x, n=n, block=64, l=l, c=c, pattern=pattern, mode=mode, scale=d ** -0.5)
    ref = orc_mod.backward(*oracle_inputs(x), pattern=pattern, mode=mode, l=l, c=c, scale=d ** -0.5)
    check_all(f"wide p{pattern} m{mode} n{n} l{l} c{c} {batch}x{heads}", got, ref, torch.bfloat16,
              names=("o", "lse", "dq", "dk", "dv"))
