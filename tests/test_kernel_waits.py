"""Hand-placed waits of the ring kernels, checked in the assembly that the build's flags give (no GPU needed): their
tiles travel by loads that the compiler does not track, so it orders nothing against them by itself."""
import os
import re
import subprocess

import pytest

from paper_2605_13784_amd import _build


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    asm = str(tmp_path_factory.mktemp("asm") / "sk_kernels.s")
    flags = [f for f in _build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + flags +
                   ["-S", "--cuda-device-only", "-o", asm, os.path.join(_build.CSRC, "sk_kernels.hip")], check=True, capture_output=True)
    with open(asm) as f:
        return f.read()


def _kernels(assembly, names):
    """(name, lines of assembly) of the kernels whose names match."""
    return [(name, [x.strip() for x in body.split("\n")])
            for name, body in re.findall(r"^(_Z\d+(?:%s)\w*):[^\n]*\n(.*?)\n\.Lfunc_end" % names, assembly, re.S | re.M)]


RING = "sk_attn_bf16_d(?:64|128)"


def test_staged_keys_are_in_memory_before_the_barrier_that_announces_them(assembly):
    """The workgroup of the own part stores a query's own K/V and then loads them into LDS, each wave tiles that others
    stored: between its last store and the next barrier every wave has to wait for its stores (vmcnt(0))."""
    found = 0
    for name, lines in _kernels(assembly, RING):
        tiles = next(i for i, x in enumerate(lines) if x.startswith("global_load_lds"))
        stores = [i for i in range(tiles) if lines[i].startswith("global_store_dwordx4")]
        assert len(stores) == 2, "%s: staging stores one K and one V piece" % name
        barrier = next(i for i in range(stores[-1], tiles) if lines[i].startswith("s_barrier"))
        assert any(x.startswith("s_waitcnt") and "vmcnt(0)" in x for x in lines[stores[-1]:barrier]), name
        found += 1
    assert found == 7


def test_partials_are_in_memory_before_the_workgroup_arrives(assembly):
    """A workgroup whose partial another one may merge in the same launch announces it by an atomic: each wave waits for its
    write-through stores (vmcnt(0)) behind the last of them, in front of the barrier and of that arrival."""
    found = 0
    for name, lines in _kernels(assembly, RING):
        arrival = next(i for i, x in enumerate(lines) if x.startswith("global_atomic_add"))
        stores = [i for i, x in enumerate(lines) if x.startswith("buffer_store_dwordx4")]
        assert stores and stores[-1] < arrival and all(lines[i].endswith("sc0 sc1") for i in stores), name
        waits = [i for i in range(stores[-1], arrival) if lines[i].startswith("s_waitcnt") and "vmcnt(0)" in lines[i]]
        assert waits and any(lines[i].startswith("s_barrier") for i in range(waits[0], arrival)), name
        found += 1
    assert found == 7


def test_weights_of_the_merge_are_written_before_the_lanes_read_them(assembly):
    """The lanes of a row exchange the weights of its parts through LDS without a barrier instruction, as they are lanes of one
    wave: the compiler is told where the writes end, and the reads of the rounds stand behind it."""
    found = 0
    for name, lines in _kernels(assembly, "sk_attn_bf16_small|sk_attn_f32"):
        at = [i for i, x in enumerate(lines) if x.startswith("; wave barrier")]
        assert len(at) == 1, name
        assert any(x.startswith("ds_write") for x in lines[at[0] - 60:at[0]]) and any(x.startswith("ds_read_b128") for x in lines[at[0]:at[0] + 60]), name
        found += 1
    assert found == 4
