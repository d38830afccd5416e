"""Checkpoints in and out (csrc/pack_transfer.cpp behind the C ABI) on a made-up GPU: host code only, compiled with
tests/transfer_driver.cpp, which defines the HIP calls, late streams and failures included.  One scenario per process."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("no hipcc to compile the driver with")
    csrc, exe = os.path.join(ROOT, "paper_2002_02885_amd", "csrc"), str(tmp_path_factory.mktemp("transfer") / "driver")
    subprocess.run([hipcc, "-x", "hip", "--cuda-host-only", "-std=c++17", "-O1", "-pthread", "-rdynamic", "-I", csrc,
                    os.path.join(csrc, "pack_api.cpp"), os.path.join(csrc, "pack_transfer.cpp"),
                    os.path.join(ROOT, "tests", "transfer_driver.cpp"), "-o", exe, "-ldl"], check=True, capture_output=True)
    return exe


def _run(driver, *args):
    r = subprocess.run([driver, *args], capture_output=True, text=True, timeout=110)
    assert r.returncode == 0 and r.stdout == "OK\n", r.stdout + r.stderr


def test_a_call_that_finds_no_pinned_memory_leaves_the_member_unchanged(driver):
    _run(driver, "no_pinned")


def test_every_kernel_of_a_transfer_is_launched_by_the_calling_thread(driver):
    """A handle may name another stream in another thread (hipStreamPerThread): weights written, a step and weights read
    back see each other, and the caller's buffer is not read after the call."""
    _run(driver, "order")


def test_transfers_with_fewer_threads_than_wanted(driver):
    _run(driver, "few_threads")


def test_a_failure_anywhere_in_a_transfer_ends_it_and_the_next_one_works(driver):
    _run(driver, "failures")


def test_a_pack_is_ready_when_the_call_that_made_it_returns(driver):
    """Creation, a joining member and a new optimiser as another thread sees them, and creation on a capturing stream."""
    _run(driver, "ready")


def test_pinned_memory_goes_with_the_last_pack(driver):
    _run(driver, "released")


def test_counted_operations_are_those_of_the_layers_without_padding(driver):
    _run(driver, "work")


def test_the_separate_update_takes_the_plain_products_and_reductions(driver):
    """A pack whose update is a launch of its own tells the kernels that produce its gradients nothing of the optimisers."""
    _run(driver, "separate_update")


def test_counted_bytes_of_the_update_follow_the_optimisers_in_force(driver):
    _run(driver, "update_bytes")


def test_products_with_few_outputs_take_larger_tiles_in_packs_of_many_members(driver):
    _run(driver, "slim_tiles")


def test_single_precision_weight_gradients_of_the_general_gather_take_larger_tiles_without_padding_to_save(driver):
    _run(driver, "gather_tiles")


def test_launch_timing_goes_on_when_a_change_of_optimiser_plans_the_launches_again(driver):
    _run(driver, "timing")


def test_a_change_of_optimiser_that_finds_no_host_memory_leaves_the_pack_unchanged(driver):
    _run(driver, "no_host_memory")
