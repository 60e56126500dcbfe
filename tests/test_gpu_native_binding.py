"""The native fast path of the Python binding against the ctypes path (taken
when `out` is given) and the Python autograd functions: the same results bit for
bit, on a current side stream too; calls that it does not take go where they
went before, with the same errors; hooks on saved tensors run."""
import pytest
import torch

from workloads import NAMES, make_gqa_inputs

pytestmark = pytest.mark.gpu

CASES = [(1, 4, 2, 130, 64, "bf16", True), (2, 3, 3, 65, 32, "f32", False), (1, 8, 1, 600, 128, "bf16", True)]


@pytest.fixture
def fb():
    import paper_2609_24089_amd as m
    m.load_library()
    return m


def tensors(case, seed=290):
    B, H, Hkv, N, d, dt, causal = case
    x = make_gqa_inputs(B, H, Hkv, N, d, dt, seed)
    return [x[n].cuda() for n in NAMES]


def through_ctypes(fb, Q, K, V, dO, UQ, UK, UV, scale, causal, use_dq=True):
    e, row = torch.empty_like, lambda: torch.empty(Q.shape[:3], device=Q.device)  # noqa: E731
    O, L = fb.attn_fwd_lse(Q, K, V, scale, causal, out=(e(Q), row()))
    dQ, dK, dV, D = fb.attn_bwd(Q, K, V, O, dO, L, scale, causal, out=(e(Q), e(K), e(K), row()))
    Qt, dOt, al, E = fb.attn_bob_pass1_rows(Q, K, V, O, dO, UQ, UK, UV, L, D, scale, causal,
                                            dQ=dQ if use_dq else None, out=(e(Q), e(Q), row(), row()))
    Kt, Vt = fb.attn_bob_pass2_cols(Q, K, V, dO, UQ, UK, UV, L, D, al, E, scale, causal, out=(e(K), e(K)))
    return dict(Qt=Qt, Kt=Kt, Vt=Vt, dOt=dOt, alpha=al, E=E, O=O, L=L, D=D, dQ=dQ, dK=dK, dV=dV)


@pytest.mark.parametrize("case", CASES, ids=str)
@pytest.mark.parametrize("use_dq", [True, False])
def test_calls_equal_the_ctypes_path(fb, case, use_dq):
    t, causal = tensors(case), case[-1]
    ref = through_ctypes(fb, *t, 0.1, causal, use_dq)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        got = fb.bob(*t, 0.1, causal=causal, use_dq=use_dq)
    side.synchronize()
    Q, K, V, dO, UQ, UK, UV = t
    assert list(got) == list(ref)
    for k in ref:
        assert torch.equal(got[k], ref[k]), k
    one = dict(zip(("O", "L"), fb.attn_fwd_lse(Q, K, V, 0.1, causal)))
    one.update(zip(("dQ", "dK", "dV", "D"), fb.attn_bwd(Q, K, V, ref["O"], dO, ref["L"], 0.1, causal)))
    one.update(zip(("Qt", "dOt", "alpha", "E"),
                   fb.attn_bob_pass1_rows(Q, K, V, ref["O"], dO, UQ, UK, UV, ref["L"], ref["D"], 0.1, causal,
                                          dQ=ref["dQ"] if use_dq else None)))
    one.update(zip(("Kt", "Vt"), fb.attn_bob_pass2_cols(Q, K, V, dO, UQ, UK, UV, ref["L"], ref["D"], ref["alpha"],
                                                        ref["E"], 0.1, causal)))
    for k in ref:
        assert torch.equal(one[k], ref[k]), k


def test_refused_calls_raise_as_before(fb):
    Q, K, V, dO, UQ, UK, UV = tensors(CASES[0])
    with pytest.raises(ValueError, match="contiguous"):
        fb.attn_fwd_lse(Q.transpose(2, 3).contiguous().transpose(2, 3), K, V, 0.1)
    with pytest.raises(ValueError, match="multiple"):
        fb.attn_fwd_lse(Q[:, :3].contiguous(), K, V, 0.1)
    with pytest.raises(TypeError, match="unsupported dtype"):
        fb.attn_fwd_lse(Q.half(), K.half(), V.half(), 0.1)
    with pytest.raises(RuntimeError, match="BOB_EUNSUPPORTED"):
        fb.attn_fwd_lse(*[x[..., :48].contiguous() for x in (Q, K, V)], 0.1)
    with pytest.raises(RuntimeError, match="BOB_EINVAL"):
        fb.attn_fwd_lse(Q, K, V, float("inf"))
    with pytest.raises(ValueError, match="ROCm device"):
        fb.bob(*[x.cpu() for x in (Q, K, V, dO, UQ, UK, UV)], 0.1)
    O, L = fb.attn_fwd_lse(Q, K, V, 0.1)
    with pytest.raises(ValueError, match="row vectors"):
        fb.attn_bwd(Q, K, V, O, dO, L.double(), 0.1)
    empty = [x[:, :, :0].contiguous() for x in (Q, K, V)]
    assert fb.attn_fwd_lse(*empty, 0.1)[0].shape == empty[0].shape


def hvp(attend, q, k, v, y, u, causal):
    O = attend(q, k, v, 0.1, causal)
    g = torch.autograd.grad(O, (q, k, v), grad_outputs=O - y, create_graph=True)
    h = torch.autograd.grad(g, (q, k, v), grad_outputs=u, retain_graph=True)
    part = torch.autograd.grad(g[1], (q, v), grad_outputs=u[1])   # two of the three cotangents undefined
    return [O, *g, *h, *part]


@pytest.mark.parametrize("case", CASES, ids=str)
def test_attention_equals_the_python_functions(fb, case):
    from paper_2609_24089_amd.autograd import _AttentionFn
    Q, K, V, dO, UQ, UK, UV = tensors(case, 291)
    q, k, v = (x.requires_grad_(True) for x in (Q, K, V))
    got = hvp(fb.attention, q, k, v, dO, (UQ, UK, UV), case[-1])
    ref = hvp(_AttentionFn.apply, q, k, v, dO, (UQ, UK, UV), case[-1])
    for i, (a, b) in enumerate(zip(got, ref)):
        assert torch.equal(a, b), i


def test_attention_under_hooks_and_transforms(fb):
    Q, K, V, dO, UQ, UK, UV = tensors(CASES[0], 292)
    q, k, v = (x.requires_grad_(True) for x in (Q, K, V))
    packed = []
    with torch.autograd.graph.saved_tensors_hooks(lambda x: packed.append(1) or x.clone(), lambda x: x):
        O = fb.attention(q, k, v, 0.1, True)
    assert len(packed) >= 4
    got = torch.autograd.grad(O, (q, k, v), grad_outputs=dO.expand_as(O))
    plain = torch.autograd.grad(fb.attention(q, k, v, 0.1, True), (q, k, v), grad_outputs=dO)
    for a, b in zip(got, plain):
        assert torch.equal(a, b)
    with pytest.raises(Exception):
        torch.func.vmap(lambda x: fb.attention(x, K.detach(), V.detach(), 0.1))(Q.detach()[None])
    with torch.autograd.forward_ad.dual_level():
        dual = torch.autograd.forward_ad.make_dual(Q.detach(), UQ)
        with pytest.raises(Exception):
            fb.attention(dual, K.detach(), V.detach(), 0.1)
    with torch.no_grad():
        assert fb.attention(q, k, v, 0.1).grad_fn is None
    q2 = q * 1
    O = fb.attention(q2, k, v, 0.1)
    q2.mul_(2)   # a saved input changed in place
    with pytest.raises(RuntimeError, match="inplace|in-place"):
        torch.autograd.grad(O, (k,), grad_outputs=dO)


class Tagged(torch.Tensor):
    """A subclass that takes part in torch's functions (by the default
    __torch_function__, which keeps the type)."""


def test_tensor_subclasses_keep_their_type(fb):
    """Outputs made like an input have its class, as on the ctypes path; a Parameter
    gives plain tensors on either."""
    t = tensors(CASES[0], 293)
    plain = fb.bob(*t, 0.1, causal=True)
    sub = [x.as_subclass(Tagged) for x in t]
    got, ref = fb.bob(*sub, 0.1, causal=True), through_ctypes(fb, *sub, 0.1, True)
    for k in ref:
        assert type(got[k]) is type(ref[k]) and torch.equal(got[k].as_subclass(torch.Tensor), plain[k]), k
    assert type(got["Qt"]) is Tagged
    assert type(fb.attention(*sub[:3], 0.1, True)) is Tagged
    q = torch.nn.Parameter(t[0])
    assert type(fb.attn_fwd_lse(q, *t[1:3], 0.1)[0]) is torch.Tensor
    O = fb.attention(q, *t[1:3], 0.1, True)
    assert type(O) is torch.Tensor and "AttentionFn" not in type(O.grad_fn).__name__   # the C++ function
    dq, = torch.autograd.grad(O, (q,), grad_outputs=t[3])
    assert torch.equal(dq, plain["dQ"])
