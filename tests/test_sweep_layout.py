"""LDS layouts and addresses of the kernels, enumerated on the CPU from the
headers the kernels are built from."""
import ctypes as C
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2207_05535_amd", "csrc")
LDS = 160 * 1024


@pytest.fixture(scope="module")
def layout(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.exists("/opt/rocm/include/hip"):
        pytest.skip("HIP headers or g++ not available")
    out = tmp_path_factory.mktemp("layout") / "layout.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", "-I" + CSRC, os.path.join(HERE, "sweep_layout.cpp"), "-o", str(out)], check=True)
    lib = C.CDLL(str(out))
    lib.sweep_lds.restype = lib.wrong_candidates.restype = lib.pairing_lds.restype = C.c_int64
    return lib


@pytest.mark.parametrize("threads", [64, 128, 256, 512, 1024])
def test_sweep_addresses_stay_in_the_lattices(layout, threads):
    """Every word a lane of the streamed sweep flips or reads lies in the
    workgroup's lattices, for every lattice size and the numbers of groups that
    fit; every unit is visited once."""
    idle = 0
    for L in list(range(4, 95, 2)) + [100, 110, 126, 128]:
        for groups in (1, 2, 3, 4, 5, 7, 16, 41, 64, 255, 256):
            if groups > 1 and (L > 64 or groups * L * L > 16384) or layout.sweep_lds(L, threads, groups, 1) > LDS:
                continue
            out = (C.c_int64 * 6)()
            layout.sweep_walk(L, threads, groups, out)
            words = groups * L * L
            assert 0 <= out[0] and out[1] < words, (L, groups, list(out))
            assert 0 <= out[2] and out[3] < words, (L, groups, list(out))
            assert out[4] == 0, (L, groups)
            idle += out[5]
    assert idle > 0


@pytest.mark.parametrize("Rc", [1, 2, 3, 31, 62, 63, 64, 65, 130])
def test_pairing_candidates_are_positions(layout, Rc):
    """Lanes of the pairing repair read positions of the population alone, at
    sizes below a wavefront too."""
    assert layout.wrong_candidates(Rc) == 0


def test_fused_resampling_layout(layout):
    """The fine prefix of the one-workgroup resampling, which is stored 16
    bytes at a time, is aligned to them behind the coarse one at every
    population size, and the largest population fits a workgroup's LDS beside
    the kernel's own 4.3 KB."""
    out = (C.c_int64 * 4)()
    for R in range(1, layout.fused_max() + 1):
        layout.fused_layout(R, out)
        assert out[1] % 16 == 0 and out[0] <= out[1] < out[2] <= out[3], R
    assert out[3] + 4400 <= LDS


def test_largest_population_paired_in_lds(layout):
    """Runs of up to 20352 replicas leave the pairing kernel the kilobyte it
    asks for beside its arrays; the next size does not."""
    assert layout.pairing_lds(20352) + 1024 == LDS < layout.pairing_lds(20353) + 1024
