"""Private memory of kernels that are bound by memory traffic or issue: what
the built library's own metadata says of them.  Spilled registers and arrays
that the compiler leaves in memory cost these kernels traffic of their own."""
import os
import re
import shutil
import subprocess

import pytest

from paper_1906_06306_amd import _lib

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{demangled name: (scratch bytes per lane, static LDS bytes)}"""
    tools = [os.path.join(LLVM, t) for t in ("llvm-objcopy", "clang-offload-bundler", "llvm-readelf")] + ["c++filt"]
    if not all(shutil.which(t) for t in tools):
        pytest.skip("no LLVM tools")
    objcopy, bundler, readelf, cxxfilt = tools
    d = tmp_path_factory.mktemp("co")
    fat, co = str(d / "fat.bin"), str(d / "gfx950.co")
    subprocess.run([objcopy, f"--dump-section=.hip_fatbin={fat}", _lib.LIB_PATH, "/dev/null"], check=True)
    subprocess.run([bundler, "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950",
                    f"--input={fat}", f"--output={co}"], check=True)
    notes = subprocess.run([readelf, "--notes", co], check=True, capture_output=True, text=True).stdout
    rows = re.findall(r"\.group_segment_fixed_size: (\d+).*?\.name: +(\S+)\s+\.private_segment_fixed_size: (\d+)",
                      notes, re.S)
    names = subprocess.run([cxxfilt], input="\n".join(r[1] for r in rows), check=True, capture_output=True,
                           text=True).stdout.split("\n")
    return {n.replace("void pic::", "").split("(pic::")[0]: (int(r[2]), int(r[0])) for n, r in zip(names, rows)}


# a pattern of demangled names, how many instantiations match
LEAN = [
    (r"k_state_copy<", 6),
    (r"k_deposit<", 9),
    (r"k_push<float, 3, true, \w+, long long, 8, ", 4),                   # the 3D shock's tiles
    (r"k_push_persistent<float, 3, true, \w+, long long, 8, true, ", 2),
]


@pytest.mark.parametrize("pattern,count", LEAN)
def test_no_private_memory(kernels, pattern, count):
    found = {n: v[0] for n, v in kernels.items() if re.match(pattern, n)}
    assert len(found) == count
    assert not any(found.values()), found


def test_state_copy_holds_no_lds(kernels):
    """The compiler moves arrays it cannot keep in registers to LDS as well."""
    assert all(v[1] == 0 for n, v in kernels.items() if n.startswith("k_state_copy<"))
