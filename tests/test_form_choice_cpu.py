"""The choice of a launch's form (csrc/fb_forms.h), built with the host compiler:
it follows the compute units that the device has."""
import ctypes
import os
import random
import shutil
import subprocess

import pytest

import paper_2609_24089_amd as fb

WRAPPER = r"""
#include "fb_forms.h"
#include <vector>
extern "C" int balanced(int64_t total, int fit, int cus) { return fb::balanced_order(total, fit, cus); }
extern "C" int kept(const int* answers, int n, int* got) {  // the answers that n reads give in turn
  std::atomic<int> known{0};
  int reads = 0;
  for (int i = 0; i < n; ++i) got[i] = fb::read_once(known, [&] { return answers[reads++]; });
  return reads;
}
extern "C" int pick(const fb::FormQuery* q, int n, const fb::Form* f) {
  switch (n) {
    case 2: return fb::pick_form(*q, {f[0], f[1]});
    case 3: return fb::pick_form(*q, {f[0], f[1], f[2]});
    case 5: return fb::pick_form(*q, {f[0], f[1], f[2], f[3], f[4]});
  }
  return -1;
}
"""


class Form(ctypes.Structure):
    _fields_ = [("blocks", ctypes.c_int), ("sets", ctypes.c_int), ("resident", ctypes.c_int), ("threads", ctypes.c_int),
                ("parts", ctypes.c_int), ("extra_us", ctypes.c_double), ("weight", ctypes.c_double)]

    def __init__(self, blocks, sets, resident, threads=256, parts=1, extra_us=0.0, weight=1.0):
        super().__init__(blocks, sets, resident, threads, parts, extra_us, weight)


class Query(ctypes.Structure):
    _fields_ = [("cus", ctypes.c_int), ("heads", ctypes.c_int64), ("N", ctypes.c_int64), ("tiles", ctypes.c_int64),
                ("causal", ctypes.c_bool), ("block_us", ctypes.c_double), ("base", ctypes.c_double),
                ("per_block", ctypes.c_double), ("narrow", ctypes.c_double), ("merge_us", ctypes.c_double),
                ("margin", ctypes.c_double)]


@pytest.fixture(scope="module")
def forms(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("forms")
    src, out = str(tmp / "forms.cpp"), str(tmp / "forms.so")
    with open(src, "w") as f:
        f.write(WRAPPER)
    csrc = os.path.join(os.path.dirname(fb.__file__), "csrc")
    subprocess.run([os.environ.get("CXX") or shutil.which("g++"), "-std=c++17", "-O1", "-Wall", "-Werror", "-fPIC",
                    "-shared", "-I", csrc, "-o", out, src], check=True)
    lib = ctypes.CDLL(out)
    lib.balanced.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_int]
    lib.pick.argtypes = [ctypes.POINTER(Query), ctypes.c_int, ctypes.c_void_p]
    return lib


def pick(lib, cus, heads, N, forms, causal=False, merge_us=0.0, margin=1.0):
    q = Query(cus, heads, N, (N + 31) // 32, causal, 0.1, 4.5, 0.45, 1.0, merge_us, margin)
    return lib.pick(ctypes.byref(q), len(forms), (Form * len(forms))(*forms))


def test_the_choice_follows_the_device(forms):
    """32 whole blocks of 128 rows: narrow blocks in sets on 256 compute units, which
    the whole blocks leave idle, and whole blocks on 32 (one each) or where the
    device is unknown."""
    f = [Form(8, 1, 2), Form(1, 8, 1)]
    assert pick(forms, 256, 8, 512, f) == 1
    assert pick(forms, 32, 8, 512, f) == 0
    assert pick(forms, 0, 8, 512, f) == 0
    # 600 whole blocks, more than fit 256 compute units at two each: no other form is weighed
    assert pick(forms, 256, 150, 512, f) == 0


def test_the_balanced_order_is_for_the_whole_device(forms):
    assert forms.balanced(1024, 2, 256) == 2
    assert forms.balanced(256, 2, 256) == 0            # one round
    assert forms.balanced(6 * 256 * 2, 2, 256) == 2    # six rounds
    assert forms.balanced(6 * 256 * 2 + 1, 2, 256) == 0
    for cus in (0, 32, 64, 128, 304):                  # a part of a device, or another one
        assert forms.balanced(1024, 2, cus) == 0


def test_a_constant_that_could_not_be_read_is_read_again(forms):
    answers, got = (ctypes.c_int * 5)(0, -1, 3, 7, 7), (ctypes.c_int * 5)()
    assert forms.kept(answers, 5, got) == 3
    assert [max(0, g) for g in got] == [0, 0, 3, 3, 3]


@pytest.mark.parametrize("threads", [256, 512, 1024])
def test_no_form_that_a_launch_cannot_take(forms, threads):
    """Problems of one 16-row block a head: the narrow form wins until its grid has
    2^32 threads, and from there on the whole form runs."""
    most = (2 ** 32 - 1) // threads
    f = [Form(4, 1, 1), Form(1, threads // 64, 4, threads=threads)]
    assert pick(forms, 256, most, 16, f) == 1
    assert pick(forms, 256, most + 1, 16, f) == 0
    f = [Form(4, 1, 1), Form(1, 1, 16, threads=1, weight=0.01)]   # 2^31 blocks
    assert pick(forms, 256, 2 ** 31 - 1, 16, f) == 1
    assert pick(forms, 256, 2 ** 31, 16, f) == 0


def test_narrower_blocks_with_the_same_sets_are_never_taken(forms):
    """Forms that are not built (worth_building() in csrc/fb_launch.h): blocks whose
    sets are those of the next wider form, both within one step of a compute unit's
    four SIMDs; and two-set 128-row blocks beside two 64-row ones a compute unit."""
    rng = random.Random(7)
    for _ in range(3000):
        heads, N = rng.randint(1, 400), int(2 ** rng.uniform(0, 16))
        causal, whole = rng.random() < 0.5, Form(4, 1, rng.choice((1, 2)))
        assert pick(forms, 256, heads, N, [whole, Form(2, 2, 1), Form(1, 2, 1)], causal) != 2
        assert pick(forms, 256, heads, N, [whole, Form(2, 1, 1), Form(1, 1, 1)], causal) == 0
        assert pick(forms, 256, heads, N, [Form(8, 1, 2), Form(4, 2, 2), Form(2, 4, 1), Form(1, 4, 1), Form(8, 2, 1)],
                    causal) != 4


def test_whole_blocks_stay_where_little_is_gained(forms):
    """Two forms of equal estimate but for what the query adds: the merge of the sets,
    the margin of the row kernels, the splits' own margin and cost."""
    f = [Form(4, 1, 1), Form(4, 2, 1)]
    assert pick(forms, 256, 64, 256, f) == 1                        # half the steps
    assert pick(forms, 256, 64, 256, f, margin=4.0) == 0
    assert pick(forms, 256, 64, 256, f, merge_us=2.0) == 0          # 8 us to merge four blocks
    assert pick(forms, 256, 64, 256, [Form(4, 1, 1), Form(4, 1, 1, parts=2, extra_us=0.5)]) == 0   # a second round of 4 us
    assert pick(forms, 256, 16, 8192, [Form(8, 1, 1), Form(8, 1, 1, parts=2, extra_us=9.0)]) == 0  # 1024 blocks fill it
    assert pick(forms, 256, 1, 8192, [Form(8, 1, 1), Form(8, 1, 1, parts=2, extra_us=9.0)]) == 1   # 64 blocks do not
