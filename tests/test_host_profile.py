"""Host side of the profiler (plans, launches, pinned memory, index arithmetic) on the CPU: tests/host_profile.cpp is the library's own
source compiled for the host, on a HIP runtime that only records what is called."""
import os
import shutil
import subprocess

import pytest

from paper_2605_04711_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_04711_amd", "csrc")


@pytest.fixture(scope="module")
def host_profile(tmp_path_factory):
    """-> function that runs one check of tests/host_profile.cpp."""
    if shutil.which("hipcc") is None or shutil.which("g++") is None:
        pytest.skip("no compiler")
    out = tmp_path_factory.mktemp("host_profile")
    obj, exe = str(out / "host_profile.o"), str(out / "host_profile")
    inc = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-g", *inc, "-c", "-o", obj,
                    os.path.join(ROOT, "tests", "host_profile.cpp")], check=True, capture_output=True, timeout=300)
    # no device code: the symbol that would hold it stays undefined
    subprocess.run(["g++", "-std=c++17", "-O1", "-no-pie", "-Wl,--unresolved-symbols=ignore-all", *inc, "-o", exe, obj,
                    os.path.join(CSRC, "baoc_risk.cpp"), "-lpthread"], check=True, capture_output=True, timeout=300)

    def run(check):
        r = subprocess.run([exe, check], capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, f"{r.returncode}\n{r.stdout}{r.stderr}"
    return run


def test_step_plans_of_large_layouts(host_profile):
    host_profile("plans")


def test_states_of_small_layouts_stay_in_the_memory_side_cache(host_profile):
    host_profile("memory")


def test_finalize_waits_before_it_reports_an_error(host_profile):
    host_profile("finalize_error")


def test_a_handle_may_outlive_the_library_s_own_objects(host_profile):
    host_profile("end_at_exit")


def test_matrix_loads_stay_inside_the_parameters(host_profile):
    host_profile("reads")


def test_one_pass_reads_every_coordinate_once_inside_its_rows(host_profile):
    host_profile("once")


def test_intervals_of_the_one_pass(host_profile):
    host_profile("once_intervals")


def test_no_kernel_spills_registers_or_uses_scratch():
    """The kernels' metadata in the built library: a zero behind every such key."""
    binding.load_library()
    with open(binding._build.LIB, "rb") as f:
        lib = f.read()
    for key in (b".private_segment_fixed_size", b".vgpr_spill_count"):
        values = [lib[i + len(key)] for i in range(len(lib)) if lib.startswith(key, i)]
        assert len(values) > 50 and set(values) == {0}, (key, values)
