"""What the host code asks of the HIP runtime, against stand-ins for its calls and for the kernel launchers (no GPU needed)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def _run(tmp_path, check):
    exe = str(tmp_path / "fake_device")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-o", exe,
                    os.path.join(HERE, "host_fake_device_driver.cpp")], check=True, capture_output=True)
    r = subprocess.run([exe, check], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "fake device ok" in r.stdout, r.stdout + r.stderr


def test_pinned_ring_slots_and_the_kernels_that_read_them(tmp_path):
    _run(tmp_path, "ring")


def test_keys_that_forks_share_are_not_read_once(tmp_path):
    _run(tmp_path, "forks")


def test_pieces_of_head_dim_64_plans_whose_lists_need_no_copy(tmp_path):
    _run(tmp_path, "pieces")


def test_short_calls_merged_in_their_launch(tmp_path):
    _run(tmp_path, "merges")


def test_lists_of_batched_calls(tmp_path):
    _run(tmp_path, "lists")
