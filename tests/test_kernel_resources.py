"""Register use of the built kernels, read from the metadata of this repository's own objects: a kernel of the predicate
tasks or of the join count's usual paths that keeps registers in scratch memory pays for it with memory traffic that no timing at one
size shows (CPU only)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2305_08872_amd import build as hip_build

TOOLS = "/opt/rocm/llvm/bin"


def _tool(name):
    path = os.path.join(TOOLS, name)
    path = path if os.path.exists(path) else shutil.which(name)
    if path is None:
        pytest.skip("no " + name)
    return path


def _kernels(obj, tmp):
    """(mangled name, bytes of scratch per lane) of every gfx950 kernel of an object built here."""
    bundle, code = os.path.join(tmp, "bundle"), os.path.join(tmp, "code")
    subprocess.check_call([_tool("llvm-objcopy"), "--dump-section", ".hip_fatbin=" + bundle, obj, os.devnull])
    subprocess.check_call([_tool("clang-offload-bundler"), "--type=o", "--unbundle", "--input=" + bundle, "--output=" + code,
                           "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"])
    notes = subprocess.check_output([_tool("llvm-readelf"), "--notes", code], text=True)
    for block in re.split(r"\n  - \.agpr_count", notes)[1:]:
        yield (re.search(r"\.name:\s+(\S+)", block).group(1),
               int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", block).group(1)))


@pytest.mark.parametrize("source", [s for s in hip_build.SOURCES
                                    if re.match(r"mmlike_(tile_|critical_f64_|valu_(discount|boost|count_gt)_)|identity_split_waves|count_i8_(stream|tile)", s)])
def test_predicate_task_kernels_keep_everything_in_registers(source, tmp_path):
    obj = os.path.join(hip_build.OBJ_DIR, os.path.splitext(source)[0] + ".o")
    if not os.path.exists(obj):
        hip_build.build()
    kernels = list(_kernels(obj, str(tmp_path)))
    assert len(kernels) >= (16 if re.match("mmlike_(tile|valu)_", source) else 4)
    assert [k for k in kernels if k[1] != 0] == []
