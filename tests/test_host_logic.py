"""Host logic of the library that no GPU is needed for, compiled from the library's own header and
run on the CPU."""
import os
import shutil
import subprocess

import pytest

from conftest import ROOT


def _build_and_run(tmp_path, name):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    exe = tmp_path / name
    src = os.path.join(ROOT, "tests", "host", name + ".hip")
    subprocess.run([hipcc, "--offload-arch=gfx950", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2605_11744_amd", "csrc"), src, "-o", str(exe)],
                   check=True, capture_output=True, timeout=600)
    return subprocess.run([str(exe)], capture_output=True, text=True, timeout=600).stdout


def _build_and_run_on_cpu(tmp_path, name):
    """A check that runs kernels of the library on the CPU (tests/host/emu)."""
    clang = shutil.which("amdclang++") or "/opt/rocm/llvm/bin/clang++"
    if not os.path.exists(clang):
        pytest.skip("clang++ of ROCm not found")
    exe = tmp_path / name
    host = os.path.join(ROOT, "tests", "host")
    subprocess.run([clang, "-O1", "-std=c++17", "-I", os.path.join(host, "emu"), "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2605_11744_amd", "csrc"), "-I", "/opt/rocm/include",
                    os.path.join(host, name + ".cpp"), "-o", str(exe)], check=True, capture_output=True, timeout=600)
    return subprocess.run([str(exe)], capture_output=True, text=True, timeout=600).stdout


def test_commit_in_one_launch_in_any_order_of_its_waves(tmp_path):
    """The append kernel that updates the counters itself, its waves in orders that the hardware takes rarely
    (every workgroup's first wave before any other, the last waves first, at random): one to four
    workgroups per head, whole segments and open ones, with and without attention views."""
    out = _build_and_run_on_cpu(tmp_path, "append_order_check")
    assert out.startswith("ok "), out
    assert int(out.split()[1]) == 192


def test_items_of_packed_batches(tmp_path):
    """The numbering of a packed batch's row blocks on the CPU: every block of every sequence once per head,
    longest first for the heads that see the whole past (up to 64 sequences), empty sequences, segments off
    the block size, and the search for a block's sequence in batches of up to 300,000."""
    out = _build_and_run_on_cpu(tmp_path, "packed_items_check")
    assert out.startswith("ok "), out
    assert int(out.split()[1]) == 99


def test_item_mapping_is_one_to_one_and_longest_first(tmp_path):
    """item_coords (the integer part of the kernels' block-index resolution) over some 10,000 launch
    shapes -- dense, packed (numbered over the padded grid), retrieved-prefix and split-prefix forms,
    every sub-group count -- maps the item indices one-to-one onto (segment, block, head, sequence, sub-group, piece), lists the
    full-history heads first and longest first, and gives the same answer with the host-prepared
    divisors as with plain divisions."""
    out = _build_and_run(tmp_path, "item_coords_check")
    assert out.startswith("ok "), out
    launches, items = (int(x) for x in out.split()[1:3])
    assert launches > 5000 and items > 10_000_000


def test_launch_divisors_are_exact(tmp_path):
    """The multiply-shift pairs the launchers prepare (FastDiv) give n / d and n % d exactly for every
    divisor up to 70000, the neighbours of every power of two, 200000 random divisors, and for each
    the edge values and random n below 2^31."""
    out = _build_and_run(tmp_path, "fastdiv_check")
    assert out.startswith("ok "), out
    assert int(out.split()[1]) > 10_000_000
