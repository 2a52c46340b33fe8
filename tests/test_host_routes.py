"""Which kernels a call launches and what it allocates, without a GPU: the library runs
on a recording stand-in for the HIP runtime (hip_recorder.cpp) that counts allocations and
records launches by name."""
import os
import shutil
import subprocess

import pytest

from paper_2012_11430_amd import _lib, build as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FP64, FP32, BF16X3, DIRECT = _lib.PRONY_FP64, _lib.PRONY_FP32, _lib.PRONY_BF16X3, _lib.PRONY_FP64_DIRECT

pytestmark = pytest.mark.skipif(not os.path.exists(B.LIB) or not shutil.which("g++"),
                                reason="needs the built library and g++")


class Result:
    def __init__(self, line):
        st, allocations, held, *self.kernels = line.split()
        self.status, self.allocations, self.held = int(st), int(allocations), int(held)


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("recorder") / "hip_recorder")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"),
                    "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "hip_recorder.cpp"), "-o", exe,
                    "-rdynamic", B.LIB, "-Wl,-rpath," + os.path.dirname(B.LIB), "-Wl,--allow-shlib-undefined"],
                   check=True)

    def run(commands):
        out = subprocess.run([exe], input="\n".join(commands) + "\n", capture_output=True, text=True, timeout=300)
        assert out.returncode == 0, out.stderr
        lines = out.stdout.splitlines()
        assert len(lines) == len(commands), out.stdout[-500:]
        return [Result(x) for x in lines]
    return run


@pytest.mark.parametrize("d_max,n_max,m_max", [(3, 10, 17), (3, 10, 18), (2, 63, 20), (3, 20, 32), (1, 300, 25),
                                               (1, 1100, 9), (3, 9, 64)])
def test_calls_within_a_reserve_allocate_nothing(recorder, d_max, n_max, m_max):
    """prony_reserve covers every single-instance call up to its bounds, not the largest
    shape alone: a workspace that grows later is freed under graphs captured before."""
    shapes = [(d, n, m) for d in range(1, d_max + 1)
              for n in sorted({1, 2, 3, 5, 8, 15, 16, 31, 255, 256, n_max - 9, n_max - 1, n_max} & set(range(1, n_max + 1)))
              for m in sorted({1, 8, 9, 15, 16, 17, 24, 25, 31, 32, m_max - 1, m_max}
                              & set(range(1, min(m_max, (n + 1) ** d) + 1)))]
    calls = [f"reserve {d_max} {n_max} {m_max}"]
    for d, n, m in shapes:
        if m <= 32:
            calls += [f"build {d} {n} {m} {prec} {flags}" for prec in (FP64, FP32, BF16X3) for flags in (0, 1)]
            calls += [f"adjoint {d} {n} {m} {prec}" for prec in (FP64, FP32)]
        calls.append(f"coeffs {d} {n} {m} 1")
    done = recorder(["create"] + calls)
    grew = [(c, r.status, r.allocations) for c, r in zip(calls[1:], done[2:]) if r.status != 0 or r.allocations]
    assert not grew, f"{len(grew)} of {len(calls) - 1}: {grew[:5]}"


@pytest.mark.parametrize("call,limit,kernel", [
    (f"adjoint 3 20 20 {FP64}", 11 << 20, "adjoint_tiles<double"),
    (f"adjoint 2 127 32 {FP64}", 22 << 20, "adjoint_tiles<double"),
    (f"build 3 12 20 {FP64} 1", 9 << 20, "pencil_tiles<double"),
    (f"build 3 9 20 {FP64} 0", 3 << 20, "pencil_tiles<double"),
    (f"factors 3 20 20 {FP64} 0", 11 << 20, "pencil_pack<double>"),
    (f"factors 2 127 32 {FP64} 1", 17 << 20, "pencil_pack<double>")])
def test_calls_whose_line_spectral_memory_cannot_be_had_run_the_tiles(recorder, call, limit, kernel):
    """The limits (bytes that may be held) are enough for the tile kernels and not for the
    line-spectral form, which runs without a limit."""
    tune = [f"tune {d} {n} {m} {FP64} 1 64" for d, n, m in ((3, 12, 20), (3, 9, 20))]   # few partial rows
    few = recorder(["create"] + tune + [f"limit {limit}", call, "destroy"])
    assert few[-2].status == 0 and few[-2].held <= limit and kernel in " ".join(few[-2].kernels), vars(few[-2])
    all_of_it = recorder(["create"] + tune + [call])[-1]
    assert all_of_it.status == 0 and all_of_it.held > limit and "spectral" in " ".join(all_of_it.kernels)


def test_factors_packed_for_the_tiles_build_and_are_released(recorder):
    done = recorder(["create", f"limit {11 << 20}", f"factors 3 20 20 {FP64} 0", "limit 1000000000", "build_factors",
                     "free_factors", "destroy"])
    assert [r.status for r in done] == [0] * 7 and done[-1].held == 0
    assert done[4].kernels[0].startswith("pencil_tiles<double") and done[4].kernels[1].startswith("pencil_finish<double")


def test_batches_leave_the_rest_of_the_memory_to_the_caller(recorder):
    """64 instances run in line-spectral form; 5000, whose transforms would take 134 GB for S
    and 86 GB for gradients, as tiles, which take 62 and 24 GB."""
    one = "3 15 32 "
    few = recorder(["create", f"batch {FP64} " + 64 * one, "run_batch", "adjoint_batch"])
    assert "spectral" in few[2].kernels[0] and "spectral" in few[3].kernels[-1]
    many = recorder(["create", f"batch {FP64} " + 5000 * one, "run_batch", "adjoint_batch", "free_batch", "destroy"])
    assert [r.status for r in many] == [0] * 6 and many[-1].held == 0
    assert many[1].held < 70e9 and "pencil_tiles_batched" in " ".join(many[2].kernels)
    assert many[3].held - many[1].held < 30e9 and "adjoint_tiles_batched" in " ".join(many[3].kernels)


@pytest.mark.parametrize("d,n,m,box", [
    (1, 447, 20, True), (1, 448, 20, False), (1, 1023, 5, False), (1, 543, 40, True), (1, 895, 64, True), (1, 896, 64, False),
    (2, 63, 20, True), (2, 119, 16, True), (2, 120, 16, False), (2, 127, 17, True), (2, 128, 17, False),
    (3, 20, 5, True), (3, 21, 5, False), (3, 24, 20, True), (3, 25, 20, False)])
def test_vandermonde_products_take_the_form_that_measured_faster(recorder, d, n, m, box):
    """Sums per axis by one workgroup a row, up to the lines and sample counts where the tiled
    launches are faster (they took half the time at d = 1, n = 1023)."""
    one, with_AT = recorder(["create", f"coeffs {d} {n} {m} 0", f"coeffs {d} {n} {m} 1"])[1:]
    tiled = ["coeffs_tiles", "coeffs_finish"]
    assert one.status == 0 and one.kernels == (["coeffs_box"] if box else tiled)
    assert with_AT.status == 0 and with_AT.kernels == tiled


@pytest.mark.parametrize("d,n,m,tiles", [
    (1, 255, 8, True), (1, 256, 8, False), (1, 255, 9, False), (1, 63, 16, True), (1, 64, 9, False), (2, 7, 8, True),
    (2, 8, 2, False), (2, 4, 16, True), (2, 5, 16, False), (3, 2, 8, True), (3, 3, 1, False), (3, 2, 16, True), (3, 2, 17, False)])
def test_small_fp64_builds_take_the_tiles(recorder, d, n, m, tiles):
    """Two launches instead of three for prepared factors, three instead of four for the first
    builds without allocation, and the same kernels in every entry point, so the same bits."""
    build, factors, prepared, fixed = recorder(
        ["create", f"build {d} {n} {m} {FP64} 0", f"factors {d} {n} {m} {FP64} 0", "build_factors"])[1:] + recorder(
        ["create", f"noalloc {d} {n} {m} {FP64} 0"])[1:]
    for r in (build, factors, prepared, fixed):
        assert r.status == 0 and any("pencil_tiles" in k or "pencil_pack" in k for k in r.kernels) == tiles, r.kernels
    assert len(prepared.kernels) == (2 if tiles else 3)
    assert len(fixed.kernels) == (3 if tiles else 4)


@pytest.mark.parametrize("d,n,m,kernels", [
    (2, 1, 4, 2), (2, 7, 32, 2), (2, 14, 32, 2), (2, 15, 2, 3), (3, 3, 20, 2), (3, 3, 21, 3), (3, 9, 4, 2), (3, 10, 1, 3)])
def test_the_smallest_fp64_gradients_take_two_launches(recorder, d, n, m, kernels):
    run = recorder(["create", f"reserve {d} {n} {m}", f"adjoint {d} {n} {m} {FP64}"])[-1]
    assert run.status == 0 and run.allocations == 0 and len(run.kernels) == kernels
    assert (run.kernels == ["adjoint_pack<double>", "adjoint_lines"]) == (kernels == 2)


def test_direct_fp64_runs_the_tiles_in_every_entry_point(recorder):
    calls = [f"build 3 9 12 {DIRECT} 1", f"noalloc 2 31 9 {DIRECT} 0", f"factors 2 31 9 {DIRECT} 0", "build_factors",
             f"adjoint 2 31 9 {DIRECT}", f"adjoint 2 3 2 {DIRECT}", f"product 3 9 4 {DIRECT} 0", f"product 2 31 1 {DIRECT} 1",
             f"batch {DIRECT} 2 31 9 3 5 4", "run_batch", "adjoint_batch"]
    done = recorder(["create"] + calls)[1:]
    assert [r.status for r in done] == [0] * len(done)
    kernels = [" ".join(r.kernels) for r in done]
    assert not any("spectral" in k or "adjoint_lines" in k or "float" in k for k in kernels)
    for k, name in zip(kernels, ["pencil_tiles<double", "pencil_tiles<double", "pencil_pack<double", "pencil_tiles<double",
                                 "adjoint_tiles<double", "adjoint_tiles<double", "toeplitz_mm_tiles<double",
                                 "toeplitz_mv<double", "", "pencil_tiles_batched<double", "adjoint_tiles_batched<double"]):
        assert name in k, (name, k)
    refused = recorder(["create", "build 2 15 5 3 0", "adjoint 2 15 5 5", f"tune 2 15 5 {DIRECT} 1 64"])[1:]
    assert [r.status for r in refused] == [_lib.PRONY_EINVAL] * 3
