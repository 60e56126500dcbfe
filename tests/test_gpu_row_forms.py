"""Every form of the row kernels (rows per workgroup, wave sets) on a problem whose
layout query names that form: the row outputs against the float64 oracle on sampled
heads, at lengths that end inside a tile, and the forward's moves of its reference
maximum (scores that keep growing along the keys, as in test_gpu_forward_rescale.py)
in the whole-block forms, whose waves hold two row blocks and share one growth check."""
import math

import pytest
import torch

import oracle
from tests.parity_util import TOL, lib, nrel, say
from tests.test_gpu_forward_rescale import late_rescales, ramp_inputs
from workloads import NAMES, as_f64, make_gqa_inputs

pytestmark = pytest.mark.gpu

DT = {"bf16": torch.bfloat16, "f32": torch.float32}
# the forms that the estimate takes (kernel: 0 forward, 1 first backward, 2 Pass 1)
FORMS = {
    (0, "bf16", 32): [(128, 1), (128, 2), (64, 4), (32, 8), (16, 16)],
    (0, "bf16", 64): [(128, 1), (128, 2), (64, 4), (32, 8), (16, 8)],
    (0, "bf16", 128): [(128, 1), (128, 2), (64, 4), (32, 4), (16, 4)],
    (0, "bf16", 256): [(64, 1), (64, 2), (32, 2)],
    (0, "f32", 32): [(64, 1), (64, 4), (32, 8), (16, 8)],
    (0, "f32", 64): [(64, 1), (64, 4), (32, 4), (16, 4)],
    (0, "f32", 128): [(64, 1), (64, 2), (32, 2)],
    (1, "bf16", 32): [(128, 1), (128, 2), (64, 4), (32, 8), (16, 16)],
    (1, "bf16", 64): [(128, 1), (128, 2), (64, 4), (32, 8), (16, 8)],
    (1, "bf16", 128): [(128, 1), (64, 2), (32, 4), (16, 4)],
    (1, "bf16", 256): [(64, 1), (64, 2), (32, 2)],
    (1, "f32", 32): [(64, 1), (64, 4), (32, 8), (16, 8)],
    (1, "f32", 64): [(64, 1), (64, 2), (32, 4), (16, 4)],
    (1, "f32", 128): [(64, 1), (64, 2), (32, 2)],
    (2, "bf16", 32): [(64, 1), (64, 2), (32, 4), (16, 8)],
    (2, "bf16", 64): [(64, 1), (64, 2), (32, 4), (16, 4)],
    (2, "bf16", 128): [(128, 1), (64, 2), (32, 2)],
    (2, "bf16", 256): [(64, 1)],
    (2, "f32", 32): [(64, 1), (64, 2), (32, 4), (16, 4)],
    (2, "f32", 64): [(64, 1), (64, 2), (32, 2)],
    (2, "f32", 128): [(64, 1)],
}
OUTS = {0: ("O", "L"), 1: ("dQ", "D"), 2: ("Qt", "dOt", "alpha", "E")}


def problem(kernel, dt, d, form, causal, least, group=1):
    """(H, N) of the least work, N >= least, that runs `form`."""
    fb = lib()
    found = []
    for N in (70, 101, 149, 200, 250, 301, 401, 523, 650, 777, 1101, 1500, 2100, 3001, 4099):
        for Hkv in (1, 2, 3, 4, 5, 6, 8, 10, 12, 14, 16, 20, 24, 28, 32, 40, 48, 56, 64, 80, 96, 128, 192, 256, 384, 512, 768):
            if N >= least and fb.row_layout(kernel, DT[dt], 1, Hkv * group, Hkv, N, d, causal) == form:
                found.append((Hkv * group * N * N, Hkv * group, N))
    assert found, "no problem runs this form"
    return min(found)[1:]


@pytest.mark.parametrize("causal", [False, True], ids=["dense", "causal"])
@pytest.mark.parametrize("kernel,dt,d,form", [(*k, f) for k, fs in FORMS.items() for f in fs], ids=str)
def test_row_form(kernel, dt, d, form, causal):
    fb = lib()
    group = 2 if causal else 1
    H, N = problem(kernel, dt, d, form, causal, 70, group)
    Hkv = H // group
    say(f"[row forms] kernel {kernel} {dt} d{d} {form}: H{H} Hkv{Hkv} N{N} causal={causal}")
    x = make_gqa_inputs(1, H, Hkv, N, d, dt, 300)
    out = fb.bob(*[x[n].cuda() for n in NAMES], d ** -0.5, causal=causal)
    for kh in sorted({0, Hkv // 2, Hkv - 1}):
        q, k = slice(kh * group, (kh + 1) * group), slice(kh, kh + 1)
        args = [as_f64(x[n][:, k if n in ("K", "V", "UK", "UV") else q]) for n in NAMES]
        ref = oracle.bob_gqa(*args, d ** -0.5, causal=causal)
        for name in OUTS[kernel]:
            a, b = as_f64(out[name][:, q]), ref[name]
            if causal and name in ("dQ", "Qt"):   # row 0 is exactly zero up to rounding
                a, b = a[:, :, 1:], b[:, :, 1:]
            assert nrel(a, b) <= TOL[dt], (name, kh, nrel(a, b))


@pytest.mark.parametrize("causal", [False, True], ids=["dense", "causal"])
@pytest.mark.parametrize("dt,d,form", [(dt, d, f) for (k, dt, d), fs in FORMS.items() if k == 0
                                       for f in fs if f[0] >= (128 if dt == "bf16" and d < 256 else 64)], ids=str)
def test_growing_row_maxima_in_whole_blocks(dt, d, form, causal):
    fb = lib()
    H, N = problem(0, dt, d, form, causal, 301)
    say(f"[row forms] growing maxima {dt} d{d} {form}: H{H} N{N} causal={causal}")
    Q, K, V = ramp_inputs(1, H, N, d, dt, 310)
    scale = 1.0 / math.sqrt(d)
    O, L = fb.attn_fwd_lse(Q.cuda(), K.cuda(), V.cuda(), scale, causal=causal)
    assert bool(torch.isfinite(O).all()) and bool(torch.isfinite(L).all())
    for h in sorted({0, H // 2, H - 1}):
        O_ref, L_ref, _, S = oracle.forward_head(*[as_f64(t[0, h]) for t in (Q, K, V)], scale, causal)
        moves = late_rescales(S)
        assert moves > N // 4, moves
        eO, eL = nrel(as_f64(O[0, h]), O_ref), nrel(as_f64(L[0, h]), L_ref)
        assert eO <= TOL[dt] and eL <= TOL[dt], (h, eO, eL)


def test_row_layout_queries():
    fb = lib()
    for kernel in (fb.BOB_ROWS_FWD, fb.BOB_ROWS_BWD, fb.BOB_ROWS_PASS1):
        assert fb.row_layout(kernel, torch.bfloat16, 1, 4, 2, 0, 64) == (0, 1)
        for bad, what in (((3, torch.bfloat16, 1, 4, 2, 9, 64), "EINVAL"), ((kernel, torch.bfloat16, 1, 4, 3, 9, 64), "EINVAL"),
                          ((kernel, torch.float32, 1, 4, 2, 9, 256), "EUNSUPPORTED")):
            with pytest.raises(RuntimeError, match=what):
                fb.row_layout(*bad)
