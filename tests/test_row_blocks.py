"""The blocks of row-broadcast multiply-adds (band_rows.h) where the caller's
values coincide: an input that has the same value as an accumulator must not
share its register, or the block's later instructions read what its first one
wrote.  Compiled for gfx950 with the library's flags; in every block of the
generated assembly no instruction may read the register that an earlier one of
the block wrote.
"""
import re
import subprocess

import pytest

from paper_1607_00693_amd import build

SOURCE = """
#include "band_rows.h"
using namespace stomsfem;
#define KERNEL(name, N, ...)                                                      \\
  extern "C" __global__ void name(double* p) {                                    \\
    double w[N], nl = p[threadIdx.x + 64 * N], f[10];                             \\
    for (int i = 0; i < N; ++i) w[i] = p[threadIdx.x + 64 * i];                   \\
    for (int i = 0; i < 10; ++i) f[i] = p[threadIdx.x + 64 * (N + 1 + i)];        \\
    __VA_ARGS__;                                                                  \\
    for (int i = 0; i < N; ++i) p[threadIdx.x + 64 * i] = w[i];                   \\
    p[threadIdx.x + 64 * N] = f[0];                                               \\
  }
"""

# kernel name -> (accumulators, the call with an input equal to an accumulator)
CALLS = {}
for n in (2, 3, 4, 7, 8, 15, 16):
    CALLS[f"update{n}_col"] = (16, f"row_updates<{16 - n}, 16>(w, w[{16 - n}], nl)")
    CALLS[f"update{n}_nl"] = (16, f"row_updates<{16 - n}, 16>(w, f[0], w[{16 - n}])")
CALLS["rhs3_f"] = (3, "f[1] = f[2] = w[0]; row_rhs3<5>(w, f, nl)")
CALLS["rhs3_nl"] = (3, "row_rhs3<5>(w, f, w[0])")
CALLS["rhs3_own_nl"] = (3, "row_rhs3_own<5>(w, w[0])")
CALLS["rhs10_z"] = (10, "for (int i = 0; i < 10; ++i) f[i] = w[0]; row_rhs10<5>(w, f, nl)")
CALLS["rhs10_c"] = (10, "row_rhs10<5>(w, f, w[0])")
CALLS["lifts3_y"] = (3, "row_lifts3(w, w[0], nl)")
CALLS["lifts3_nl"] = (3, "row_lifts3(w, f[0], w[0])")


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    d = tmp_path_factory.mktemp("row_blocks")
    src, out = d / "blocks.hip", d / "blocks.s"
    src.write_text(SOURCE + "".join(f"KERNEL({k}, {n}, {call})\n" for k, (n, call) in CALLS.items()))
    r = subprocess.run([build.HIPCC, *build.CFLAGS, "--cuda-device-only", "-S", str(src), "-o", str(out)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return out.read_text()


def registers(operand):
    """Numbers of the vector registers of an operand: v[4:5] or v4."""
    m = re.fullmatch(r"v\[(\d+):(\d+)\]|v(\d+)", operand)
    if not m:
        return set()
    return {int(m[3])} if m[3] else set(range(int(m[1]), int(m[2]) + 1))


@pytest.mark.parametrize("name", sorted(CALLS))
def test_no_block_reads_what_it_wrote(assembly, name):
    body = re.search(rf"^{name}:(.*?)s_endpgm", assembly, re.S | re.M)[1]
    blocks = re.findall(r"#ASMSTART(.*?)#ASMEND", body, re.S)
    count = 0
    for block in blocks:
        written = set()
        for line in block.splitlines():
            ops = re.match(r"\s*v_fmac_f64_dpp (\S+), (\S+), (\S+) ", line)
            if not ops:
                continue
            count += 1
            # the accumulator itself (and, where it is the broadcast value, its own copy) is read before it is written
            assert not (registers(ops[2]) | registers(ops[3])) & written, block
            written |= registers(ops[1])
    assert count >= 2
