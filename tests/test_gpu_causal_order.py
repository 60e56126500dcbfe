"""Causal grids of more than one round over the compute units run their blocks
in a balanced order (heaviest first over all heads, dealt to the compute units
in alternating direction); a single head's grid runs one head after another.
The order must lose no block: every head of a many-head problem equals the same
head computed alone, the column outputs bit for bit (unsplit, in one wave set,
from the same row state, so that each sum has the same order) and the row
outputs up to the rounding of the sums, whose order may follow the grid."""
import pytest
import torch

from tests.parity_util import nrel
from workloads import NAMES, as_f64, make_gqa_inputs

pytestmark = pytest.mark.gpu

CASES = [
    # H, Hkv, N, d, dtype: blocks of 64 and 128 rows, head counts that are and are not multiples of 8
    (19, 19, 2113, 64, "bf16"),   # 17 and 34 blocks a head, a partial last round on every XCD
    (24, 6, 1500, 128, "bf16"),   # heads in groups, whole runs of heads per XCD
    (21, 7, 1000, 32, "bf16"),
    (9, 9, 2100, 256, "bf16"),
    (13, 13, 1400, 64, "f32"),
    (24, 24, 721, 128, "f32"),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"H{c[0]}kv{c[1]}N{c[2]}d{c[3]}{c[4]}")
def test_order_changes_no_result(case):
    import paper_2609_24089_amd as fb
    H, Hkv, N, d, dt = case
    G = H // Hkv
    x = {k: v.cuda() for k, v in make_gqa_inputs(1, H, Hkv, N, d, dt, 260).items()}
    one = fb.ColumnOpts(1, 1, 0)
    whole = fb.bob(*[x[n] for n in NAMES], d ** -0.5, causal=True, columns=one)
    for kh in (0, Hkv // 2, Hkv - 1):
        part = [x[n][:, kh:kh + 1] if n in ("K", "V", "UK", "UV") else x[n][:, kh * G:(kh + 1) * G] for n in NAMES]
        alone = fb.bob(*[t.contiguous() for t in part], d ** -0.5, causal=True, columns=one)
        tol = 1e-2 if dt == "bf16" else 1e-5
        for k, v in alone.items():
            got = whole[k][:, kh:kh + 1] if k in ("dK", "dV", "Kt", "Vt") else whole[k][:, kh * G:(kh + 1) * G]
            assert nrel(as_f64(got), as_f64(v)) <= tol, (k, kh)
        rows = [whole[k][:, kh * G:(kh + 1) * G].clone() for k in ("L", "D", "alpha", "E")]
        Q, K, V, dO, UQ, UK, UV = [t.contiguous() for t in part]
        Kt, Vt = fb.attn_bob_pass2_cols(Q, K, V, dO, UQ, UK, UV, *rows, d ** -0.5, True, columns=one)
        assert torch.equal(Kt, whole["Kt"][:, kh:kh + 1]) and torch.equal(Vt, whole["Vt"][:, kh:kh + 1]), kh
