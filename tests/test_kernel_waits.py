"""Hand-placed waits of the ring kernels, checked in the assembly that the build's flags give (no GPU needed): their
tiles travel by loads that the compiler does not track, so it orders nothing against them by itself."""
import os
import re
import subprocess

from paper_2605_13784_amd import _build


def test_staged_keys_are_in_memory_before_the_barrier_that_announces_them(tmp_path):
    """The workgroup of the own part stores a query's own K/V and then loads them into LDS, each wave tiles that others
    stored: between its last store and the next barrier every wave has to wait for its stores (vmcnt(0))."""
    asm = str(tmp_path / "sk_kernels.s")
    flags = [f for f in _build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + flags +
                   ["-S", "--cuda-device-only", "-o", asm, os.path.join(_build.CSRC, "sk_kernels.hip")], check=True, capture_output=True)
    found = 0
    for name, body in re.findall(r"^(_Z\d+sk_attn_bf16_d(?:64|128)\w*):[^\n]*\n(.*?)\n\.Lfunc_end", open(asm).read(), re.S | re.M):
        lines = [x.strip() for x in body.split("\n")]
        tiles = next(i for i, x in enumerate(lines) if x.startswith("global_load_lds"))
        stores = [i for i in range(tiles) if lines[i].startswith("global_store_dwordx4")]
        assert len(stores) == 2, "%s: staging stores one K and one V piece" % name
        barrier = next(i for i in range(stores[-1], tiles) if lines[i].startswith("s_barrier"))
        assert any(x.startswith("s_waitcnt") and "vmcnt(0)" in x for x in lines[stores[-1]:barrier]), name
        found += 1
    assert found == 7
