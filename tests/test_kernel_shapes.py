"""Compile-time properties of the kernels' tile shapes, checked by the compiler
on the kernels' own headers (host pass only; no GPU)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def compiles(tmp_path, source):
    from paper_1604_08501_amd import build as B
    src = tmp_path / "shapes.hip"
    src.write_text(source)
    r = subprocess.run([B.hipcc(), *B.HIPCC_FLAGS, "--offload-host-only", "-fsyntax-only", str(src)],
                       capture_output=True, text=True, timeout=300)
    return r.returncode == 0, r.stderr[-3000:]


EVEN = """
#define SEM_REAL double
#include "{inc}"
static_assert(__alignof__(semk::kPowTables) % 16 == 0, "the tables are read 16 bytes at a time");
#define CHECK(NQ) static_assert(({at}) % 2 == 0, "Nq = " #NQ);
CHECK(2) CHECK(3) CHECK(4) CHECK(5) CHECK(6) CHECK(7) CHECK(8) CHECK(9) CHECK(10)
"""


@pytest.mark.parametrize("inc,at", [
    ("rhs.inc", "semk::RhsShape<double, NQ>::TABLES"),
    ("rhs.inc", "semk::RhsShape<double, NQ, semk::FEW>::TABLES"),
    ("surface.inc", "semk::SurfShape<double, NQ>::TABLES"),
    ("sem_lines.hpp", "semk::line_tile_tables<double, NQ, 1, 5, 1>()"),
    ("sem_lines.hpp", "semk::line_tile_tables<double, NQ, 1, 8, 3>()"),
])
def test_power_tables_lie_on_16_bytes(tmp_path, inc, at):
    """The FP64 power's tables are copied to LDS 16 bytes at a time, behind a
    tile's other values: their offset in 8-byte values has to be even (it is
    odd by itself where an odd number of arrays has an odd node count)."""
    ok, err = compiles(tmp_path, EVEN.format(inc=inc, at=at))
    assert ok, err
