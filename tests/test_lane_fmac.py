"""The lane-broadcast multiply-adds (lanes.h) are several instructions in one
asm statement: no sum may share a register with the broadcast value or the
multiplier, which later instructions still read.  Compiled here for gfx950 with
sums that hold the same values as both, where only the statement's own
constraints keep them apart; the generated assembly is read back (no GPU)."""
import os
import re
import subprocess

import pytest

from paper_2101_01763_amd import build

SRC = """
#include "lanes.h"
using namespace spand;
#define KERNEL(NAME, T, N, CALL) \\
  extern "C" __global__ void NAME(T *o, const T *i) { \\
    const T h = i[threadIdx.x], p = i[threadIdx.x + 64]; \\
    T s[N]; \\
    for (int k = 0; k < N; ++k) s[k] = T(0); \\
    s[0] = h; \\
    s[1] = p; \\
    CALL; \\
    for (int k = 0; k < N; ++k) o[threadIdx.x * N + k] = s[k]; \\
  }
KERNEL(lo32, float, 8, (fmac8<0>(s, p, h)))
KERNEL(hi32, float, 8, (fmac8<8>(s, p, h)))
KERNEL(lo64, double, 8, (fmac8<0>(s, p, h)))
KERNEL(hi64, double, 8, (fmac8<8>(s, p, h)))
KERNEL(mid32, float, 4, (fmac4(s, p, h)))
KERNEL(mid64, double, 4, (fmac4(s, p, h)))
"""


def _regs(x):
    m = re.fullmatch(r"v\[(\d+):(\d+)\]", x)
    return set(range(int(m[1]), int(m[2]) + 1)) if m else {int(x[1:])}


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    d = tmp_path_factory.mktemp("lanes")
    (d / "k.hip").write_text(SRC)
    cmd = [build._hipcc(), *build.FLAGS, "-I", build.CSRC, "--offload-device-only", "-S", "-o", str(d / "k.s"),
           str(d / "k.hip")]
    subprocess.run(cmd, check=True, capture_output=True, env={**os.environ, "LC_ALL": "C"})
    return (d / "k.s").read_text()


@pytest.mark.parametrize("name,n,lanes", [("lo32", 8, range(8)), ("hi32", 8, range(8, 16)), ("lo64", 8, range(8)),
                                          ("hi64", 8, range(8, 16)), ("mid32", 4, range(4, 8)),
                                          ("mid64", 4, range(4, 8))])
def test_sums_keep_their_own_registers(assembly, name, n, lanes):
    body = assembly.split(f"\n{name}:")[1].split("s_endpgm")[0]
    ops = re.findall(r"v_fmac_f(\d\d)_dpp (v\S+), (v\S+), (v\S+) row_newbcast:(\d+)", body)
    assert [int(o[4]) for o in ops] == list(lanes) and {o[0] for o in ops} == {name[-2:]}
    dst = [_regs(o[1]) for o in ops]
    src = set().union(*(_regs(o[2]) | _regs(o[3]) for o in ops))
    assert len(set().union(*dst)) == sum(map(len, dst)) and not src & set().union(*dst)
