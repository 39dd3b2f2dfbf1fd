"""What the compiler gave the kernels of the built library, read from the code objects' own metadata: the
kernels named here keep their working set in registers.  (One with scratch sends it to device memory
and back for every row; nothing else in the tests would show that.)"""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2605_29843_amd import harp

READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"


def code_objects(path):
    """The gfx950 code objects of the bundles in a library built from several sources."""
    blob = open(path, "rb").read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = blob.find(magic)
    while at >= 0:
        pos = at + len(magic)
        (count,) = struct.unpack_from("<Q", blob, pos)
        pos += 8
        for _ in range(count):
            off, size, nlen = struct.unpack_from("<QQQ", blob, pos)
            name = blob[pos + 24:pos + 24 + nlen].decode()
            pos += 24 + nlen
            if "gfx950" in name and size:
                yield blob[at + off:at + off + size]
        at = blob.find(magic, at + 1)


@pytest.fixture(scope="module")
def scratch_bytes(tmp_path_factory):
    """{mangled kernel name: bytes of scratch per lane}"""
    if not os.path.exists(READELF):
        pytest.skip("llvm-readelf is not installed")
    out, folder = {}, tmp_path_factory.mktemp("objects")
    for i, obj in enumerate(code_objects(harp.LIB_PATH)):
        path = folder / f"{i}.co"
        path.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for kernel in re.split(r"\n\s+- \.", notes):
            name = re.search(r"\.name:\s+(_Z\S*harp\S*)", kernel)
            size = re.search(r"private_segment_fixed_size:\s+(\d+)", kernel)
            if name and size:
                out[name.group(1)] = int(size.group(1))
    assert len(out) > 100, "the library's kernels were not found"
    return out


@pytest.mark.parametrize("kernel", ["harp_grad_bwd_run_kernel", "harp_grad_fwd_run_kernel", "harp_grad_bwd_kernel", "harp_grad_pair_bwd_kernel", "harp_grad_pair_fwd_kernel",
                                    "harp_grad_lead_bwd_kernel", "harp_grad_big_bwd_kernel", "harp_grad_pair_reduce_kernel",
                                    "harp_colpair_kernel", "harp_colwide_kernel", "harp_col_one_kernel"])
def test_no_scratch(scratch_bytes, kernel):
    sizes = {k: v for k, v in scratch_bytes.items() if kernel in k}
    assert sizes
    assert not {k: v for k, v in sizes.items() if v}


def test_scratch_of_the_chain_kernels(scratch_bytes):
    """Tiles of eight rows of a chain with a last radix of 4 hold two blocks of 16 coordinates per wave and may spill a few
    registers, and so may float32 rows of a last radix of 7 with a radix-4 stage above; no other instance does."""
    sizes = {k: v for k, v in scratch_bytes.items() if "harp_chain_kernel" in k}
    assert len(sizes) > 100
    for name, size in sizes.items():   # <in, out, last radix, transposed, four rows each, stage above>
        arg = re.search(r"harp_chain_kernelI[ft](?:[ft]|S\w*_)Li(\d)ELb(\d)ELi(\d)ELi(\d)EE", name)
        assert arg, name
        r4, trn, four, top = (int(a) for a in arg.groups())
        most = 0
        if four == 2 and r4 == 4:
            most = 160 if trn else 64
        elif four == 2 and r4 == 7 and top == 4 and "kernelIff" in name:
            most = 16
        assert size <= most, (name, size)
