"""Automatic part counts of column blocks of 128 to 1023 streamed iterations:
the call runs the layout the query reports, equals the forced part count bit
for bit and the oracle within the tolerance; the allocation-free Pass 2 keeps
such blocks unsplit."""
import numpy as np
import pytest
import torch

import oracle
from tests.parity_util import TOL, nrel, say
from workloads import NAMES, as_f64, make_gqa_inputs

pytestmark = pytest.mark.gpu

CASES = [
    # B, H, Hkv, N, d, dtype, causal
    (1, 8, 1, 513, 128, "bf16", True),    # 8 heads x 17 tiles = 136 iterations per block
    (1, 8, 1, 512, 64, "bf16", False),    # exactly 128
    (1, 8, 1, 480, 64, "bf16", False),    # 120: below the floor
    (1, 12, 2, 700, 32, "f32", True),     # 132
    (1, 4, 1, 1027, 256, "bf16", True),   # 132, one wave per SIMD when split
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"H{c[1]}kv{c[2]}N{c[3]}d{c[4]}{c[5]}{'causal' if c[6] else ''}")
def test_short_blocks(case):
    import paper_2609_24089_amd as fb
    B, H, Hkv, N, d, dt, causal = case
    iters = H // Hkv * -(-N // 32)
    x = make_gqa_inputs(B, H, Hkv, N, d, dt, 270)
    xd = {k: v.cuda() for k, v in x.items()}
    tdt = torch.bfloat16 if dt == "bf16" else torch.float32
    lays = [fb.column_layout(k, tdt, B, H, Hkv, N, d, causal)[0] for k in (fb.BOB_COLUMNS_BWD, fb.BOB_COLUMNS_PASS2)]
    say(f"[short blocks] {case}: {iters} iterations, layouts {lays}")
    assert all(lay.parts >= 2 if iters >= 128 else lay.parts == 1 for lay in lays)
    scale = d ** -0.5
    out = fb.bob(*[xd[n] for n in NAMES], scale, causal=causal)
    ref = oracle.bob_gqa(*[as_f64(x[n]) for n in NAMES], scale, causal=causal)
    for k in ("dK", "dV", "Kt", "Vt"):
        assert nrel(as_f64(out[k]), ref[k]) <= TOL[dt], k
    for lay, keys in zip(lays, (("dK", "dV"), ("Kt", "Vt"))):
        if lay.parts > 1:
            forced = fb.bob(*[xd[n] for n in NAMES], scale, causal=causal, columns=fb.ColumnOpts(lay.parts, 0, 0))
            for k in keys:
                assert torch.equal(out[k], forced[k]), k
    args = [xd[n] for n in ("Q", "K", "V", "dO", "UQ", "UK", "UV")] + [out[n] for n in ("L", "D", "alpha", "E")]
    got = fb.attn_bob_pass2_cols_noalloc(*args, scale, causal)
    want = fb.attn_bob_pass2_cols(*args, scale, causal, columns=fb.ColumnOpts(1, 0, 0))
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
