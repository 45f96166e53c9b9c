"""Direct-to-LDS loads take their LDS address from m0 and their base from scalar
registers, and need a wait state after a write of m0 and five after a vector
instruction wrote the base.  The compiler adds none for an asm block, so the built code
is looked at."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1904_10509_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

KERNEL = """
#include "sa_tile.h"
__global__ void tiles(const uint16_t* x, const float* s, float* out, int n) {
    __shared__ uint16_t t[4][64 * 64];
    __shared__ float r[64];
    sa::TileLoader<64, 64, 4> ld;
    ld.init(64, __builtin_amdgcn_readfirstlane(threadIdx.x / 64), threadIdx.x % 64);
    ld.issue(x, sa::lds_addr(&t[0][0]));
    ld.issue_rows(x, sa::lds_addr(&t[1][0]), 64, n, threadIdx.x % 64);
    ld.issue_halves(x, x + 4096, sa::lds_addr(&t[2][0]));
    sa::load_row_stats_async(s, n, sa::lds_addr(r), threadIdx.x % 64);
    sa::wait_loads_upto<0>();
    __syncthreads();
    out[threadIdx.x] = t[threadIdx.x & 3][threadIdx.x] + r[threadIdx.x & 63];
}
"""


def listing(path, out):
    subprocess.run([HIPCC, "-O3", "-std=c++17", "--offload-arch=gfx950", "--cuda-device-only", "-S", "-I", CSRC, str(path),
                    "-o", str(out)], check=True, capture_output=True)
    return [line.split(";")[0].strip() for line in open(out)]


def wait_states(code, i):
    """Wait states right before instruction i, up to the last vector one or write of m0."""
    n, m0 = 0, None
    for x in reversed(code[:i]):
        if re.match(r"v_", x) or x.endswith(":"):
            return n, m0
        if m0 is None and re.match(r"s_\w+ m0\b", x):
            m0 = n
        n += int(x.split()[1], 0) + 1 if x.startswith("s_nop") else 1
    return n, m0


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
@pytest.mark.parametrize("source", [None, os.path.join(ROOT, "paper_1904_10509_amd", "probe", "dma_read.hip")])
def test_wait_states_before_the_load(tmp_path, source):
    if source is None:
        source = tmp_path / "tiles.hip"
        source.write_text(KERNEL)
    code = [x for x in listing(source, tmp_path / "k.s") if x and not x.startswith((".p", ".s", "#"))]
    loads = [i for i, x in enumerate(code) if x.startswith("global_load_lds_dword")]
    assert loads
    for i in loads:
        vector, m0 = wait_states(code, i)
        assert m0 >= 1 and vector >= 5, code[i - 6:i + 1]
