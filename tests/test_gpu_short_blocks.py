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


@pytest.mark.parametrize("dt,H,Hkv,N,d,causal", [("bf16", 8, 1, 1024, 128, True), ("f32", 6, 2, 700, 128, False)])
def test_no_workspace_or_asked_wave_sets_run_unsplit(dt, H, Hkv, N, d, causal):
    """Blocks whose automatic layout splits: a C caller without a workspace (or with
    one that is too small or misaligned) gets the unsplit layout, and so does a
    request for wave sets; a forced part count still needs its workspace."""
    import ctypes
    import paper_2609_24089_amd as fb
    lib = fb.load_library()
    code = fb.BOB_BF16 if dt == "bf16" else fb.BOB_F32
    tdt = torch.bfloat16 if dt == "bf16" else torch.float32
    x = {k: v.cuda() for k, v in make_gqa_inputs(1, H, Hkv, N, d, dt, 271).items()}
    scale, one = d ** -0.5, fb.ColumnOpts(1, 0, 0)
    ref = fb.bob(*[x[n] for n in NAMES], scale, causal=causal, columns=one)
    for kernel in (fb.BOB_COLUMNS_BWD, fb.BOB_COLUMNS_PASS2):
        assert fb.column_layout(kernel, tdt, 1, H, Hkv, N, d, causal)[0].parts > 1
        for sets in (1, 2):
            asked = fb.column_layout(kernel, tdt, 1, H, Hkv, N, d, causal, fb.ColumnOpts(0, sets, 0))
            assert asked[0].parts == 1 and asked[1] == 0
            if sets == 1:
                assert asked[0].wave_sets == 1
    p = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    head = (code, 1, H, Hkv, N, d, ctypes.c_float(scale), int(causal))
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    small = torch.empty(64, dtype=torch.uint8, device="cuda")
    large = torch.empty(8 * 2 * Hkv * N * d * 4 + 16, dtype=torch.uint8, device="cuda")
    for ws, nbytes in ((None, 0), (p(small), 64), (ctypes.c_void_p(large.data_ptr() + 8), large.numel() - 8)):
        Kt, Vt = torch.empty_like(x["K"]), torch.empty_like(x["K"])
        mats = [p(x[n]) for n in ("Q", "K", "V", "dO", "UQ", "UK", "UV")] + [p(ref[n]) for n in ("L", "D", "alpha", "E")]
        call = lambda o: lib.attn_bob_pass2_cols_gqa_ws(*head, *mats, p(Kt), p(Vt), o, ws, nbytes, stream)  # noqa: E731
        assert call(None) == fb.BOB_OK
        assert torch.equal(Kt, ref["Kt"]) and torch.equal(Vt, ref["Vt"])
        assert call(ctypes.byref(fb.ColumnOpts(8, 0, 0))) == fb.BOB_EINVAL
        outs = [torch.empty_like(x["Q"]), torch.empty_like(x["K"]), torch.empty_like(x["K"]), torch.empty_like(ref["D"])]
        mats = [p(x[n]) for n in ("Q", "K", "V")] + [p(ref["O"]), p(x["dO"]), p(ref["L"])]
        call = lambda o: lib.attn_bwd_gqa_ws(*head, *mats, *map(p, outs), o, ws, nbytes, stream)  # noqa: E731
        assert call(None) == fb.BOB_OK
        for got, k in zip(outs, ("dQ", "dK", "dV", "D")):
            assert torch.equal(got, ref[k]), k
        assert call(ctypes.byref(fb.ColumnOpts(8, 0, 0))) == fb.BOB_EINVAL
