"""Every kernel of the library is compiled in one translation unit: a kernel that
several units hold has one host symbol for copies that may be built with different
flags, and link order decides which of them runs."""
import collections
import re
import subprocess

from tests.test_wait_states_cpu import code_objects, llvm_tool


def kernels(obj):
    out = subprocess.run([llvm_tool("llvm-readelf"), "--symbols", "--wide", obj], check=True, capture_output=True,
                         text=True).stdout
    return set(re.findall(r"\s(\S+)\.kd$", out, flags=re.M))


def test_each_kernel_is_in_one_unit(tmp_path):
    where = collections.defaultdict(list)
    for i, obj in enumerate(code_objects(str(tmp_path))):
        for k in kernels(obj):
            where[k].append(i)
    assert len(where) > 100
    several = {k: v for k, v in where.items() if len(v) > 1}
    assert not several, (len(several), sorted(several.items())[:3])
