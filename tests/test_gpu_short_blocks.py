"""Automatic layouts of column blocks of fewer than 1024 streamed iterations:
split over workgroups, narrow blocks in several wave sets, or whole blocks, by
estimated time.  The call equals the layout that the query reports, forced, bit for
bit, and the oracle within the tolerance (lengths around one block and one tile,
fewer tiles than sets, grouped heads, every head dim and both types); the
allocation-free Pass 2 keeps such blocks unsplit."""
import numpy as np
import pytest
import torch

import oracle
from tests.parity_util import TOL, nrel, say
from workloads import NAMES, as_f64, make_gqa_inputs

pytestmark = pytest.mark.gpu

SIZES = [  # B, H, Hkv, N, causal
    (1, 1, 1, 1, False),
    (1, 2, 1, 17, True),
    (1, 1, 1, 33, False),
    (2, 3, 3, 65, True),
    (1, 4, 2, 250, False),
    (1, 8, 1, 513, True),    # 136 iterations in few blocks: split
    (3, 8, 4, 389, True),
]
KEYS = ("dK", "dV", "Kt", "Vt")


@pytest.mark.parametrize("dt,d", [("bf16", 32), ("bf16", 64), ("bf16", 128), ("bf16", 256), ("f32", 32), ("f32", 64),
                                  ("f32", 128)])
@pytest.mark.parametrize("size", SIZES, ids=lambda s: f"B{s[0]}H{s[1]}kv{s[2]}N{s[3]}{'causal' if s[4] else ''}")
def test_short_blocks(size, dt, d):
    import paper_2609_24089_amd as fb
    B, H, Hkv, N, causal = size
    x = make_gqa_inputs(B, H, Hkv, N, d, dt, 270)
    xd = {k: v.cuda() for k, v in x.items()}
    tdt = torch.bfloat16 if dt == "bf16" else torch.float32
    lays = [fb.column_layout(k, tdt, B, H, Hkv, N, d, causal)[0] for k in (fb.BOB_COLUMNS_BWD, fb.BOB_COLUMNS_PASS2)]
    say(f"[short blocks] {size} {dt} d{d}: layouts {lays}")
    scale = d ** -0.5
    out = fb.bob(*[xd[n] for n in NAMES], scale, causal=causal)
    ref = oracle.bob_gqa(*[as_f64(x[n]) for n in NAMES], scale, causal=causal)
    for k in KEYS:
        a, b = as_f64(out[k]), ref[k]
        if np.linalg.norm(b) < 1e-6 * np.sqrt(b.size):   # N = 1: zero outputs
            assert np.abs(a).max() <= (0.1 if dt == "bf16" else 1e-5), k
        else:
            assert nrel(a, b) <= TOL[dt], (k, nrel(a, b))
    for lay, keys in zip(lays, (("dK", "dV"), ("Kt", "Vt"))):
        if lay.parts > 1 or lay.wave_sets > 1:
            want = fb.ColumnOpts(lay.parts, 0 if lay.parts > 1 else lay.wave_sets, 0)
            forced = fb.bob(*[xd[n] for n in NAMES], scale, causal=causal, columns=want)
            for k in keys:
                assert torch.equal(out[k], forced[k]), k
    args = [xd[n] for n in ("Q", "K", "V", "dO", "UQ", "UK", "UV")] + [out[n] for n in ("L", "D", "alpha", "E")]
    got = fb.attn_bob_pass2_cols_noalloc(*args, scale, causal)
    want = fb.attn_bob_pass2_cols(*args, scale, causal, columns=fb.ColumnOpts(1, 0, 0))
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


def test_splits_where_blocks_are_few():
    import paper_2609_24089_amd as fb
    for dt, H, Hkv, N, d, causal in ((torch.bfloat16, 8, 1, 1024, 128, True), (torch.float32, 6, 2, 700, 128, False)):
        lay, nbytes = fb.column_layout(fb.BOB_COLUMNS_PASS2, dt, 1, H, Hkv, N, d, causal)
        say(f"[short blocks] H{H} Hkv{Hkv} N{N} d{d}: {lay}, {nbytes} bytes")
        assert lay.parts >= 4 and nbytes == lay.parts * 2 * Hkv * N * d * 4
