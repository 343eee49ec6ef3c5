"""include/lattice.h stands alone: it compiles by itself as C and as C++, with warnings
as errors, whatever a program includes before it."""
import os
import subprocess

import pytest

INCLUDE = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include")


@pytest.mark.parametrize("compiler,std,suffix", [("gcc", "c99", "c"), ("g++", "c++17", "cpp")])
def test_header_compiles_alone(tmp_path, compiler, std, suffix):
    src = tmp_path / f"alone.{suffix}"
    src.write_text('#include "lattice.h"\nint main(void) { return sizeof(lat_stats) == 0; }\n')
    r = subprocess.run([compiler, f"-std={std}", "-pedantic", "-Wall", "-Werror", "-I", INCLUDE, "-c", str(src), "-o",
                        str(tmp_path / "alone.o")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
