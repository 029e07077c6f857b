"""Size rules of the dispatch that no GPU test can reach (populations of many GB),
compiled for the host from the library's own header."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "native", "dispatch_sizes.cpp")
CSRC = os.path.join(ROOT, "paper_0905_2441_amd", "csrc")


@pytest.fixture(scope="module")
def answers(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("native") / "dispatch_sizes")
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-I", CSRC,
                    "-I", os.path.join(ROOT, "include"), "-o", exe, SRC],
                   check=True, capture_output=True)

    def ask(lines):
        out = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True,
                             check=True).stdout
        return [tuple(int(v) for v in line.split()) for line in out.strip().splitlines()]
    return ask


def test_fp64_matrix_form_leaves_sizes_beyond_its_launches_to_the_valu_form(answers):
    """A grid has fewer than 2^32 threads: one per particle and component in the
    proposals, four per particle (of whole tiles of 64) in the partial sums."""
    cases = [(8, 1, 1), (8, 16384, 1), (8, 2 ** 28, 1), (8, 2 ** 29 - 32, 1), (8, 2 ** 29 - 31, 0),
             (8, 2 ** 29, 0), (4, 2 ** 30 - 64, 1), (4, 2 ** 30, 0), (2, 2 ** 30 - 64, 1),
             (2, 2 ** 30 - 63, 0), (1, 2 ** 30 - 64, 1), (1, 2 ** 30 - 63, 0), (1, 2 ** 31 - 1, 0)]
    got = answers([f"fits {k} {N}" for k, N, _ in cases])
    assert got == [(w,) for _, _, w in cases]


def test_proposal_threads_are_numbered_beyond_2_31(answers):
    """N * k = 2^31 and more (k = 8, N = 2^28): every thread has its particle and
    component, and the first one past the end has none."""
    cases = [(0, 2 ** 28, 8, (1, 0, 0)), (2 ** 31 - 1, 2 ** 28, 8, (1, 2 ** 28 - 1, 7)),
             (2 ** 31, 2 ** 28, 8, (0, -1, -1)), (2 ** 31, 2 ** 28 + 1, 8, (1, 2 ** 28, 0)),
             (2 ** 32 - 257, 2 ** 29 - 32, 8, (1, 2 ** 29 - 33, 7)),
             (2 ** 32 - 256, 2 ** 29 - 32, 8, (0, -1, -1)), (14, 5, 3, (1, 4, 2)), (15, 5, 3, (0, -1, -1))]
    got = answers([f"column {q} {N} {k}" for q, N, k, _ in cases])
    assert got == [w for *_, w in cases]


@pytest.mark.parametrize("kd", [1, 2, 4, 8])
@pytest.mark.parametrize("slices", [1, 2, 4, 16])
def test_move_lds_leaves_a_cu_its_waves(answers, kd, slices):
    """At any N (up to 1024 CDF chunks) a move's workgroup takes no more LDS than the
    ancestor search and the move need one after the other, and the random numbers of
    several moves leave room for the 16 waves a CU that the registers admit (or one
    move's numbers, the least)."""
    chunks = [0, 1, 128, 256, 512, 1024]
    got = answers([f"lds {slices} {c} {kd} 10" for c in chunks])
    for c, (one, many, batch) in zip(chunks, got):
        search = 8 * (3 * c + 256) if c else 0
        row = 512 * slices                           # 64 doubles, a row of a wave each
        assert one == max(512 * (2 * kd + 2) + 2 * row, search)
        work = 512 * (kd + 1) * (batch + 1) + 2 * row
        assert many == max(work, search) and one < 65536 and many < 65536
        assert 1 <= batch <= 10
        assert batch == 1 or (160 * 1024) // work * slices >= 16


def test_fp64_matrix_form_leaves_short_data_to_the_valu_form(answers):
    """Short data, where the VALU form's single launches (several moves in one, the
    chain of steps) are faster."""
    cases = [(1, 191, 64, 1, 0), (1, 192, 64, 1, 1), (2, 50, 65536, 1, 0), (2, 192, 65536, 1, 1),
             (4, 63, 8193, 1, 0), (4, 63, 8192, 1, 1), (4, 64, 65536, 1, 1), (8, 1, 65536, 1, 1),
             (2, 63, 8193, 0, 0), (2, 64, 8193, 0, 1), (4, 31, 8192, 0, 0), (4, 32, 8192, 0, 1),
             (8, 15, 8193, 0, 0), (8, 15, 8192, 0, 1), (8, 16, 8193, 0, 1)]
    got = answers([f"pays {k} {n} {N} {m}" for k, n, N, m, _ in cases])
    assert got == [(w,) for *_, w in cases]
