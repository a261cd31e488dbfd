"""The library's host code (dispatch, launch sizes, workspaces) over a HIP
runtime of the host alone: the sources are compiled for the host only and
linked with tests/native/fake_hip.h, which counts allocations, frees and
waits and keeps a list of the launches.  No GPU, and no device code."""
import concurrent.futures as cf
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_1705_08213_amd", "csrc")


@pytest.fixture(scope="module")
def host_check(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    from paper_1705_08213_amd.build import SOURCES
    tmp = tmp_path_factory.mktemp("host")
    srcs = [os.path.join(CSRC, s) for s in SOURCES] + [os.path.join(HERE, "native", "host_check.cpp")]

    def compile_one(src):
        obj = str(tmp / (os.path.basename(src) + ".o"))
        r = subprocess.run([hipcc, "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-x", "hip",
                            "-I", os.path.join(ROOT, "include"), "-c", src, "-o", obj],
                           capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        return obj

    with cf.ThreadPoolExecutor(max_workers=8) as ex:
        objs = list(ex.map(compile_one, srcs))
    exe = str(tmp / "host_check")
    # the device code of the sources, which is not there, is never looked at
    r = subprocess.run(["g++", "-no-pie", *objs, "-o", exe, "-lpthread", "-ldl",
                        "-Wl,--unresolved-symbols=ignore-in-object-files"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]

    def run(scenario, **env):
        out = subprocess.run([exe, scenario], capture_output=True, text=True, timeout=120,
                             env=dict(os.environ, **env))
        assert out.returncode == 0 and out.stdout.startswith("ok"), out.stdout + out.stderr
    return run


def test_launches_stay_within_the_runtime_limits(host_check):
    """No launch of 2^32 or more work-items along a dimension, whatever the
    sizes: a selection of 400,000 rows and 1000 fields is 19.5 million 64 x 64
    tiles of 256 threads."""
    host_check("launch_limits")


def test_captured_calls_have_workspaces_of_their_own(host_check):
    """Two captures on one stream, the forks of a capture and the stream's eager
    calls all have their own workspaces, and a capture's stay allocated."""
    host_check("captures")


def test_operands_without_room_cost_nothing(host_check):
    """On a nearly full card calls read the packed rows without a wait, a failed
    allocation or another stream's buffers given back."""
    host_check("nearly_full")


def test_operands_held_are_bounded(host_check):
    """Twelve streams of 3.3 GB and six batches of 1 GB hold 16 GiB at most."""
    host_check("held")


def test_forty_streams_in_turn_wait_for_nothing(host_check):
    """More streams than a framework's pool has: no waits and no allocations
    after the first round; a thousand streams wait once in 64."""
    host_check("many_streams")


def test_tile_shapes_by_form_and_size(host_check):
    """Selections, tables alone, rectangles and accumulating calls leave the
    32 x 32 tiles earlier than dense triangles with CCC rows do."""
    host_check("shapes")


def test_streamed_tables_of_complete_data(host_check):
    """Rectangles whose rows start on multiples of 64 bytes stream their tables
    from shorter fields on than other outputs."""
    host_check("streamed_tables")


def test_small_triples_rule(host_check):
    """Two turns of the chip take the general 3-way kernel alone only while the
    fields are not long."""
    host_check("small_triples")


def test_large_calls_on_long_fields_read_packed_rows(host_check):
    """Past 1,864,135 fields only the field-split tiles are exact on operands;
    calls of 3000 of them and more read the packed rows."""
    host_check("long_fields")


def test_row_ranges_lay_out_their_own_rows(host_check):
    """Rows before a range's first tile are counted, not laid out."""
    host_check("row_ranges")


def test_blocks_with_shared_counts_add_one_side_after_the_other(host_check):
    """Two sides that share count entries are not added to by one launch, whose
    workgroups would race on them."""
    host_check("shared_counts")


def test_batches_under_different_operand_limits(host_check):
    """Limits that differ past 32 bits are different batches."""
    host_check("batch_limits")


def test_forced_splits(host_check):
    """The environment's split of a tile's fields takes 1 to 64 and ignores
    anything else."""
    host_check("forced_splits")
