"""Strided heads whose stride is a multiple of the block size: the blocks away from
the band are single diagonals, whose probabilities and score gradients stay in
fp32 (rank-1 steps), where a matrix product would take them in bf16.

The bar is in units of the rounding of the bf16 result itself, |bf16(ref) - ref| in
the 2-norm.  With fp32 diagonals little is added to it: by the blocks on and next to
the diagonal, whose probabilities enter their products in bf16, and, in dQ and dK, by
the rounded O in D = dO . O.  Probabilities rounded to bf16 throughout add an error of
about the same size again.  Measured over these cases, fp32 | bf16: O 1.03 to 1.10 |
1.15 to 1.24, dV 1.10 to 1.18 | 1.34 to 1.42, dQ and dK 1.19 to 1.23 | 1.45 to 1.50
merged, 1.25 to 1.43 | 1.57 to 1.68 in A2 alone (fewer keys a row)."""
import pytest
import torch

from oracle import oracle as orc_mod
from paper_1904_10509_amd import sparse_attn as sa
from paper_1904_10509_amd.inputs import make_inputs

from gpu_util import oracle_inputs, run_gpu

pytestmark = pytest.mark.gpu

S = sa.SA_STRIDED
A2, MG, IL = sa.SA_MODE_A2, sa.SA_MODE_MERGED, sa.SA_MODE_INTERLEAVED


def excess(got, ref):
    """Error of a bf16 result over the rounding of the exact one."""
    ref = torch.from_numpy(ref)
    rounding = (ref.to(torch.bfloat16).double() - ref).norm()
    return float((torch.from_numpy(got) - ref).norm() / rounding)


# (mode, n, B, l, d, batch, heads): n / l is no multiple of 16, or l does not divide n
@pytest.mark.parametrize("mode,n,B,l,d,batch,heads", [
    (A2, 2560, 64, 64, 64, 1, 2),
    (A2, 2624, 64, 128, 64, 1, 3),
    (A2, 2592, 32, 32, 128, 1, 1),
    (IL, 2560, 64, 64, 64, 1, 4),
    (IL, 3072, 64, 64, 128, 1, 2),
    (MG, 2064, 16, 16, 64, 1, 2),
    (MG, 2576, 16, 16, 128, 1, 1),
    (MG, 4112, 16, 16, 32, 1, 2),
])
def test_far_diagonals_stay_in_fp32(mode, n, B, l, d, batch, heads):
    x = make_inputs(batch, heads, n, d, torch.bfloat16, seed=n + l + d)
    got = run_gpu(x, n=n, block=B, l=l, c=0, pattern=S, mode=mode, scale=d ** -0.5)
    ref = orc_mod.backward(*oracle_inputs(x), pattern=S, mode=mode, l=l, c=0, scale=d ** -0.5)
    first, step = (1, 2) if mode == IL else (0, 1)  # the heads with A2
    over = {name: excess(got[name][:, first::step], ref[name][:, first::step]) for name in ("o", "dq", "dk", "dv")}
    print(f"precision m{mode} n{n} B{B} l{l} d{d}: " + ", ".join(f"{k} {v:.3f}" for k, v in over.items()), flush=True)
    grad = 1.33 if mode == MG else 1.5
    assert over["o"] <= 1.125 and over["dv"] <= 1.25 and over["dq"] <= grad and over["dk"] <= grad, over
