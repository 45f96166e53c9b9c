"""Strided heads by band and residue classes or in one pass where the classes do not
fill their blocks (l not dividing n, or n / l not a multiple of the class block), l
does not fit the block grid, and heads alternate, and the same where B divides l and
the block path stays: against the fp64 oracle."""
import pytest
import torch

from oracle import oracle as orc_mod
from paper_1904_10509_amd import sparse_attn as sa
from paper_1904_10509_amd.inputs import make_inputs

from gpu_util import check_all, device, oracle_inputs, run_gpu, to64

pytestmark = pytest.mark.gpu

S = sa.SA_STRIDED
A1, A2, MG, IL = sa.SA_MODE_A1, sa.SA_MODE_A2, sa.SA_MODE_MERGED, sa.SA_MODE_INTERLEAVED

# (mode, n, B, l, d, batch, heads)
CASES = [
    (MG, 512, 64, 100, 64, 1, 2),     # 5 or 6 positions per class
    (MG, 1024, 64, 37, 64, 2, 3),     # 27 or 28, l < B
    (MG, 1536, 32, 47, 128, 1, 2),    # 32 or 33: some classes end one block earlier
    (MG, 1600, 64, 49, 32, 1, 1),     # 32 or 33, one (batch, head)
    (MG, 2048, 16, 31, 64, 1, 2),     # 66 or 67
    (MG, 3072, 64, 24, 64, 1, 2),     # 128 exactly, l < B
    (MG, 2064, 16, 16, 128, 1, 2),    # 129, B divides l: the block path
    (MG, 1552, 16, 12, 128, 1, 1),    # 129 or 130
    (MG, 1168, 16, 12, 128, 2, 1),    # 97 or 98
    (MG, 4112, 16, 16, 64, 1, 2),     # 257, B divides l
    (MG, 2000, 16, 3, 32, 1, 2),      # 666 or 667
    (MG, 3072, 64, 128, 128, 2, 2),   # 24, B divides l
    (MG, 832, 64, 64, 64, 1, 2),      # 13, B divides l
    (MG, 1024, 64, 64, 64, 6, 8),     # 16: 192 workgroups of the one-pass forward, its smallest
    (MG, 1024, 64, 64, 64, 1, 47),    # 188: band and classes apart
    (A2, 1008, 16, 50, 64, 1, 2),     # 20 or 21
    (A2, 1088, 64, 130, 64, 2, 2),    # 8 or 9
    (A2, 2000, 16, 7, 128, 1, 1),     # 285 or 286
    (A2, 2320, 16, 24, 128, 1, 1),    # 96 or 97: past one launch per class at d = 128
    (A2, 3104, 16, 24, 64, 1, 2),     # 129 or 130: past one launch per class
    (A2, 6160, 16, 24, 64, 1, 1),     # 256 or 257: class blocks of 64, a last block of one
    (A2, 2048, 16, 24, 32, 2, 1),     # 85 or 86 in one launch
    (IL, 1024, 64, 64, 64, 2, 4),     # B divides l: the block path
    (IL, 992, 32, 45, 64, 1, 5),      # an odd number of heads
    (IL, 992, 32, 45, 128, 2, 3),     # odd and batched: the classes' heads make no one index
    (IL, 1280, 64, 30, 32, 1, 1),     # no odd head
    (A1, 1024, 64, 100, 64, 2, 2),
    (A1, 448, 64, 1 << 30, 64, 1, 1),
    (MG, 448, 64, 1 << 30, 32, 1, 1),
]


@pytest.mark.parametrize("mode,n,B,l,d,batch,heads", CASES)
def test_band_and_classes(mode, n, B, l, d, batch, heads):
    x = make_inputs(batch, heads, n, d, torch.bfloat16, seed=n + l % 1000 + d)
    got = run_gpu(x, n=n, block=B, l=l, c=0, pattern=S, mode=mode, scale=d ** -0.5)
    ref = orc_mod.backward(*oracle_inputs(x), pattern=S, mode=mode, l=l, c=0, scale=d ** -0.5)
    check_all(f"classes m{mode} n{n} B{B} l{l} d{d} {batch}x{heads}", got, ref, torch.bfloat16,
              names=("o", "lse", "dq", "dk", "dv"))


@pytest.mark.parametrize("mode,l", [(MG, 45), (A2, 45), (IL, 45)])
def test_stages_and_neighbours(mode, l):
    """The backward's stages one by one, in views of larger buffers whose other
    elements stay untouched (padding rows of a class are never written)."""
    dev = device()
    n, B, d, b, h = 992, 32, 64, 1, 4
    x = make_inputs(b, h, n, d, torch.bfloat16, seed=77)
    lay = sa.build_layout(n, B, l, 0, S, mode, device=dev)

    def view(src=None):
        """[b, h, n, d] inside [b, h, n + 2, d] filled with 5, the outermost rows outside the view."""
        buf = torch.full((b, h, n + 2, d), 5.0, dtype=torch.bfloat16, device=dev)
        if src is not None:
            buf[:, :, 1:n + 1] = src.to(dev)
        return buf, buf[:, :, 1:n + 1]

    (_, q), (_, k), (_, v), (_, dout) = (view(x[name]) for name in ("q", "k", "v", "dout"))
    outs = [view() for _ in range(4)]
    o, lse = sa.forward(q, k, v, lay, out=outs[0][1])
    grads = tuple(t for _, t in outs[1:])
    ws = torch.empty(sa.sparse_attn_bwd_workspace_size(*lay.pattern_args, b, h, d, sa.SA_BF16) + 64, dtype=torch.uint8,
                     device=dev)
    for stage in (sa.SA_BWD_ROW_STATS, sa.SA_BWD_DQ, sa.SA_BWD_DKDV):
        sa.backward(q, k, v, o, dout, lse, lay, grads=grads, workspace=ws, stages=stage)
    torch.cuda.synchronize()
    ref = orc_mod.backward(*oracle_inputs(x), pattern=S, mode=mode, l=l, c=0, scale=d ** -0.5)
    got = {name: to64(t) for name, t in zip(("o", "dq", "dk", "dv"), (o,) + grads)}
    check_all(f"stages m{mode} l{l}", dict(got, lse=to64(lse)), ref, torch.bfloat16, names=("o", "lse", "dq", "dk", "dv"))
    for buf, _ in outs:
        assert bool((buf[:, :, 0] == 5).all()) and bool((buf[:, :, n + 1] == 5).all())
