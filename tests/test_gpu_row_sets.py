"""GPU parity of the row kernels' small-grid forms (16, 32 or 64 query rows per
workgroup, the streamed key tiles dealt to several wave sets whose sums meet in
LDS) against the float64 oracle: lengths around one row block and one tile, with
fewer tiles than wave sets (sets without a tile), with row blocks past the
diagonal of the last tile, grouped heads, every head dim and both types.  Rows
whose maximum lies in one set only check the merge of the forward's references."""
import numpy as np
import pytest
import torch

import oracle
from tests.parity_util import TOL, nrel, say
from workloads import NAMES, as_f64, make_gqa_inputs

pytestmark = pytest.mark.gpu

ROW_OUTS = ("O", "L", "D", "dQ", "Qt", "dOt", "alpha", "E")
SIZES = [  # B, H, Hkv, N, causal
    (1, 1, 1, 1, False),
    (1, 2, 1, 17, True),
    (1, 1, 1, 33, False),
    (2, 3, 3, 65, True),
    (1, 4, 2, 250, False),
    (1, 2, 2, 517, True),
    (3, 8, 4, 389, True),    # more blocks than compute units in the narrow forms
]


def zero_tol(dt, d):
    """Largest value of an output that is exactly zero: scale (a - b) K, where a
    and b are equal sums of d products of N(0, 1) values (of size sqrt(d)) in two
    orders.  In fp32 each sum is off by about u d (d steps of u sqrt(d), added as a
    random walk), the scale is 1 / sqrt(d), K is at most 4, and E's part has two such
    sums with a factor alpha of about 1.5: 32 u sqrt(d) in all.  In bf16 the inputs
    of the products carry 8 bits: 0.1, as for the column outputs."""
    return 0.1 if dt == "bf16" else 32 * 2.0 ** -24 * d ** 0.5


@pytest.mark.parametrize("dt,d", [("bf16", 32), ("bf16", 64), ("bf16", 128), ("bf16", 256), ("f32", 32), ("f32", 64),
                                  ("f32", 128)])
@pytest.mark.parametrize("size", SIZES, ids=lambda s: f"B{s[0]}H{s[1]}kv{s[2]}N{s[3]}{'causal' if s[4] else ''}")
def test_row_forms(size, dt, d):
    import paper_2609_24089_amd as fb
    B, H, Hkv, N, causal = size
    x = make_gqa_inputs(B, H, Hkv, N, d, dt, 280)
    scale = d ** -0.5
    out = fb.bob(*[x[n].cuda() for n in NAMES], scale, causal=causal)
    ref = oracle.bob_gqa(*[as_f64(x[n]) for n in NAMES], scale, causal=causal)
    for k in ROW_OUTS:
        a, b = as_f64(out[k]), ref[k]
        if causal and k == "Qt":   # row 0 is exactly zero up to one bf16 rounding
            a, b = a[:, :, 1:], b[:, :, 1:]
        if np.linalg.norm(b) < 1e-6 * np.sqrt(max(1, b.size)):   # N = 1: zero outputs
            assert np.abs(a).max(initial=0.0) <= zero_tol(dt, d), (k, np.abs(a).max())
            continue
        assert nrel(a, b) <= TOL[dt], (k, nrel(a, b))


@pytest.mark.parametrize("dt,d", [("bf16", 64), ("bf16", 128), ("f32", 64)])
@pytest.mark.parametrize("at", [0, 100, 299])
def test_forward_sets_of_unequal_reference(dt, d, at):
    """One key dominates every row by far more than the forward's rescale
    threshold, so the wave set that streams it has a far higher reference than
    the others, whose sums must vanish in the merge."""
    import paper_2609_24089_amd as fb
    x = make_gqa_inputs(1, 2, 2, 300, d, dt, 281)
    x["Q"][..., 0] = 4.0
    x["K"][:, :, at, 0] = 64.0
    say(f"[row sets] dominating key {at} {dt} d{d}")
    O, L = fb.attn_fwd_lse(x["Q"].cuda(), x["K"].cuda(), x["V"].cuda(), 1.0)
    ref = oracle.bob_gqa(*[as_f64(x[n]) for n in NAMES], 1.0)
    assert torch.isfinite(L).all()
    assert nrel(as_f64(O), ref["O"]) <= TOL[dt] and nrel(as_f64(L), ref["L"]) <= 1e-5
