"""An infinity or a NaN reaches the rows that attend it and no others: rows of K and
V at one position, or of Q and dO, are poisoned, and every result that does not
depend on them is compared with the fp64 oracle on the clean inputs."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc_mod
from paper_1904_10509_amd import sparse_attn as sa
from paper_1904_10509_amd.inputs import make_inputs

from gpu_util import check, check_lse, device, oracle_inputs, to64

pytestmark = pytest.mark.gpu

S, F, P = sa.SA_STRIDED, sa.SA_FIXED, sa.SA_FIXED_PER_HEAD
A1, A2, MG, IL = sa.SA_MODE_A1, sa.SA_MODE_A2, sa.SA_MODE_MERGED, sa.SA_MODE_INTERLEAVED
NAMES = ("q", "k", "v", "dout")


def attended(pattern, mode, n, l, c, h):
    """S as a matrix [i, j] (Sec. 4.3, 5.1) for head h."""
    i, j = np.arange(n)[:, None], np.arange(n)[None, :]
    if pattern == S:
        a1, a2 = i - j <= l, (i - j) % l == 0
    else:
        w = l - (h % (l // c) + 1) * c if pattern == P else l - c
        a1, a2 = i // l == j // l, (j % l >= w) & (j % l < w + c)
    part = (A1, A2)[h % 2] if mode == IL else mode
    return (j <= i) & (a1 if part == A1 else a2 if part == A2 else a1 | a2)


def poisoned(x, names, at, value):
    """The inputs with the rows `at` of the named tensors all value (alternating in sign where infinite)."""
    out = dict(x)
    for name in names:
        t = x[name].clone()
        t[:, :, at] = value
        if not np.isnan(value):
            t[:, :, at, 1::2] = -value
        out[name] = t
    return out


def run_poisoned(pattern, mode, n, B, l, c, d, dtype, batch, heads, at, value, backward=True, only=None):
    dev = device()
    x = make_inputs(batch, heads, n, d, dtype, seed=n + l + d)
    scale = d ** -0.5
    ref = orc_mod.backward(*oracle_inputs(x), pattern=pattern, mode=mode, l=l, c=c, scale=scale)
    lay = sa.build_layout(n, B, l, c, pattern, mode, device=dev)
    clean = {name: x[name].to(dev) for name in NAMES}
    o, lse = sa.forward(clean["q"], clean["k"], clean["v"], lay, scale)
    keys = {name: t.to(dev) for name, t in poisoned(x, ("k", "v"), at, value).items()}
    rows = {name: t.to(dev) for name, t in poisoned(x, ("q", "dout"), at, value).items()}
    o1, lse1 = sa.forward(keys["q"], keys["k"], keys["v"], lay, scale)
    grads1 = grads2 = None
    if backward:
        grads1 = sa.backward(keys["q"], keys["k"], keys["v"], o, keys["dout"], lse, lay, scale)
        grads2 = sa.backward(rows["q"], rows["k"], rows["v"], o, rows["dout"], lse, lay, scale)
    torch.cuda.synchronize()
    for h in range(heads):
        if only is not None and mode == IL and (A1, A2)[h % 2] != only:
            continue  # (the band's blocks multiply a block's neighbours too)
        own = attended(pattern, mode, n, l, c, h)
        free = ~own[:, at].any(axis=1)  # rows that attend no poisoned key
        far = ~own[at].any(axis=0)      # keys that no poisoned row attends
        other = ~np.isin(np.arange(n), at)
        label = f"{value} at {at} p{pattern} m{mode} n{n} B{B} l{l} d{d} head {h}"
        pick = lambda t, keep: to64(t)[:, h][:, keep]  # noqa: E731
        check(f"{label} o", pick(o1, free), ref["o"][:, h][:, free], dtype)
        check_lse(f"{label} lse", pick(lse1, free), ref["lse"][:, h][:, free], dtype)
        if not backward:
            continue
        check(f"{label} dq (keys)", pick(grads1[0], free), ref["dq"][:, h][:, free], dtype)
        check(f"{label} dq (rows)", pick(grads2[0], other), ref["dq"][:, h][:, other], dtype)
        check(f"{label} dk", pick(grads2[1], far), ref["dk"][:, h][:, far], dtype)
        check(f"{label} dv", pick(grads2[2], far), ref["dv"][:, h][:, far], dtype)


# (pattern, mode, n, B, l, c, d, heads, poisoned positions)
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("pattern,mode,n,B,l,c,d,heads,at", [
    (S, A1, 64, 16, 64, 0, 32, 1, [9, 40]),       # dense: the future of rows before 9
    (S, MG, 160, 32, 12, 0, 64, 2, [0, 77]),
    (S, A2, 192, 64, 24, 0, 128, 1, [100]),
    (F, MG, 256, 64, 48, 10, 64, 2, [150, 63]),
    (F, IL, 192, 32, 64, 16, 32, 2, [70, 127]),
    (P, A2, 192, 16, 40, 10, 128, 2, [55]),
])
def test_f32(pattern, mode, n, B, l, c, d, heads, at, value):
    run_poisoned(pattern, mode, n, B, l, c, d, torch.float32, 1, heads, at, value)


# the one-pass kernels: a chunk reaches up to 31 rows, in a class 31 l positions, past
# the last attended one
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("n,B,l,d,batch,heads,at", [
    (1024, 64, 37, 64, 2, 2, [700, 41]),
    (1536, 32, 47, 128, 1, 2, [1000, 1535]),
    (1600, 64, 49, 32, 1, 1, [3, 900]),
    (3072, 64, 24, 64, 1, 1, [2047]),
    (1024, 64, 64, 64, 6, 8, [600]),    # filled classes: one pass in the forward alone
])
def test_one_pass(n, B, l, d, batch, heads, at, value):
    run_poisoned(S, MG, n, B, l, 0, d, torch.bfloat16, batch, heads, at, value, backward=l % B != 0)


# the residue classes (A2 alone, the odd ones of alternating heads): one launch per
# class, separate launches, padded and whole class blocks
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("mode,n,B,l,d,heads,at", [
    (A2, 1008, 16, 50, 64, 2, [600, 20]),
    (A2, 1088, 64, 130, 32, 1, [700]),
    (A2, 2000, 16, 7, 128, 1, [1000]),
    (A2, 4096, 32, 32, 64, 1, [2000, 4095]),
    (A2, 4112, 16, 12, 64, 1, [1999]),
    (IL, 992, 32, 45, 64, 4, [500]),
    (IL, 1280, 64, 30, 128, 2, [700]),
])
def test_classes(mode, n, B, l, d, heads, at, value):
    run_poisoned(S, mode, n, B, l, 0, d, torch.bfloat16, 1, heads, at, value, only=A2)
