"""The built library's kernels hold no function calls (CPU: the code objects' symbols): a call in a
kernel first waits for every load in flight, and the network's kernels are written to have all of a
layer chain's weights in flight before the first product."""
import os
import re
import subprocess

import pytest

from test_kernel_resources import LIB, TARGET, _tool


def test_kernels_call_no_device_functions(tmp_path):
    tools = [_tool(t) for t in ("llvm-objcopy", "clang-offload-bundler", "llvm-readelf")]
    if not os.path.exists(LIB) or not all(tools):
        pytest.skip("library or LLVM tools not available")
    objcopy, bundler, readelf = tools
    fat = tmp_path / "fatbin"
    subprocess.run([objcopy, "--dump-section", f".hip_fatbin={fat}", LIB, str(tmp_path / "copy.so")], check=True,
                   capture_output=True)
    data = fat.read_bytes()
    starts = [m.start() for m in re.finditer(re.escape(b"__CLANG_OFFLOAD_BUNDLE__"), data)]
    kernels, others = set(), set()
    for i, s in enumerate(starts):
        part, co = tmp_path / f"b{i}", tmp_path / f"b{i}.co"
        part.write_bytes(data[s:starts[i + 1] if i + 1 < len(starts) else len(data)])
        if subprocess.run([bundler, "--unbundle", "--type=o", "--input", str(part), f"--targets={TARGET}", "--output",
                           str(co)], capture_output=True).returncode != 0:
            continue
        table = subprocess.run([readelf, "--symbols", "--wide", str(co)], capture_output=True, text=True, check=True).stdout
        names = {f[-1]: f[3] for f in (line.split() for line in table.splitlines()) if len(f) >= 8 and f[0][:-1].isdigit()}
        functions = {n for n, kind in names.items() if kind == "FUNC"}
        kernels |= {n for n in functions if n + ".kd" in names}
        others |= {n for n in functions if n + ".kd" not in names}
    assert len(kernels) >= 60
    assert not others, others
