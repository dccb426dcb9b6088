"""The scratch of the Coulomb and exchange builds against what their plans write, on the
host: tests/native/jk_scratch.cpp is compiled against csrc/kernels.h, linked with
the built library, and sweeps the plan functions that the launches use (no GPU call)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1707_03771_amd")


@pytest.fixture(scope="module")
def sweep(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("native") / "jk_scratch")
    subprocess.run(["g++", "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(PKG, "csrc"),
                    os.path.join(ROOT, "tests", "native", "jk_scratch.cpp"), "-o", exe, "-L" + PKG, "-ldfx",
                    "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath," + PKG, "-Wl,-rpath,/opt/rocm/lib"], check=True)

    def run(what):
        r = subprocess.run([exe, what], capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stdout + r.stderr
        return int(r.stdout)
    return run


def test_coulomb_plans_stay_inside_their_scratch(sweep):
    """With fewer tiles kept the rounded number of parts can be larger (33 of 36 tiles: 7
    parts of gamma, 36: 6), so a build must not be cut by rounding alone."""
    assert sweep("coulomb") > 1_000_000


def test_density_exchange_scratch_holds_both_signs(sweep):
    """A build of fewer columns can want more partial sums, so the scratch of an indefinite
    density's two builds is not that of the larger count."""
    assert sweep("exchange") > 100_000


def test_fit_workspace_counts_padded_rows_and_lists(sweep):
    """Raw's rows are whole 128-byte lines, so up to 15 doubles longer than its columns."""
    assert sweep("fit") == 128
