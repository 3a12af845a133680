"""Host side of lattices, batches and pools, without a GPU: libfhp.so runs over a stand-in
for the HIP runtime (native/hip_standin.h), which shows every launch and what
its tables hold."""
import os
import shutil
import subprocess

import pytest

from paper_1208_2428_amd import _binding as B

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = "/opt/rocm"


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    if not shutil.which("g++") or not os.path.isdir(os.path.join(ROCM, "include", "hip")):
        pytest.skip("g++ or the HIP headers are not available")
    if not os.path.exists(B.lib_path()):
        from paper_1208_2428_amd import build
        build.build()
    exe = str(tmp_path_factory.mktemp("host") / "batch_host_check")
    lib = os.path.abspath(B.lib_path())
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-rdynamic", "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(ROCM, "include"), os.path.join(HERE, "native", "batch_host_check.cpp"),
                    lib, "-Wl,-rpath," + os.path.dirname(lib), "-Wl,-rpath," + os.path.join(ROCM, "lib"),
                    "-Wl,--allow-shlib-undefined", "-o", exe], check=True)

    def run(name):
        r = subprocess.run([exe, name], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0 and r.stdout.startswith("OK"), (r.returncode, r.stdout, r.stderr)
    return run


def test_tiles_are_launched_over_tile_tables(check):
    """A tiling set between tiled steps, or a call of no steps, leaves bands in
    the tables' memory: the next tiled step has to build its own again."""
    check("retile")


def test_repeated_calls_write_no_tables(check):
    """Steps after steps of one kind leave the tables and the host alone."""
    check("repeat")


def test_routes_by_shape(check):
    """Bands for one pass over even members and enough rounds, else tiles."""
    check("routes")


def test_waves_of_a_tile(check):
    """Waves with words in a launch over many lattices: those the shapes count."""
    check("waves")


def test_ticks_run_what_the_host_counts(check):
    """Jobs of every remainder, ended ones kept resident, one to five passes a tick."""
    check("jobs")


def test_an_upload_starts_with_its_copy(check):
    """No kernel is queued in front of a state's first chunk."""
    check("upload")


def test_short_calls(check):
    """Two and three steps: a sweep at the edges of where it fills the device,
    tiles beyond them."""
    check("shallow")


def test_bands_of_tall_lattices(check):
    """Passes of two and four steps over narrow rows."""
    check("tall")
