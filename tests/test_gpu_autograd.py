"""attention(): the C++ node and the Python node are the same function - results, gradients, refusals,
hooks on saved tensors - and what the C++ node does not take still reaches the Python node."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _qkv(B, H, Hkv, Nq, Nk, d, layout, seed=0):
    g = torch.Generator().manual_seed(seed)
    def one(h, n):
        if layout == "fused":
            return torch.randn((B, n, 3, h, d), generator=g).to(torch.bfloat16).to(DEV)
        t = torch.randn((B, n, h, d), generator=g).to(torch.bfloat16).to(DEV).permute(0, 2, 1, 3)
        return t.contiguous() if layout == "bhnd" else t
    if layout == "fused":
        x = one(H, Nq)
        return [x[:, :, i].permute(0, 2, 1, 3) for i in range(3)]
    return [one(H, Nq), one(Hkv, Nk), one(Hkv, Nk)]


CASES = [(2, 3, 3, 100, 100, 64, "bhnd"), (2, 3, 3, 128, 128, 64, "bnhd"), (1, 2, 2, 130, 130, 96, "fused"),
         (1, 4, 2, 65, 65, 128, "bhnd"), (1, 4, 2, 65, 65, 32, "bnhd"), (1, 2, 2, 33, 200, 64, "bhnd"), (1, 1, 1, 1100, 1100, 64, "bhnd")]


@pytest.mark.parametrize("case", CASES, ids=str)
@pytest.mark.parametrize("variant", [0, 1, 2])
def test_both_nodes_agree(lib, case, variant):
    from paper_2510_04212_amd import autograd as A
    data = _qkv(*case)
    do = torch.randn(data[0].shape, generator=torch.Generator().manual_seed(5)).to(torch.bfloat16).to(DEV)
    out = []
    for node in ("c++", "python"):
        q, k, v = (t.detach().requires_grad_(True) for t in data)
        if node == "c++":
            o = A.attention(q, k, v, True, 0.1, variant)
            assert "CppNode" in o.grad_fn.name()
        else:
            o = A._FlashAttention.apply(q, k, v, True, 0.1, variant, None, None)
        out.append((o.detach(),) + torch.autograd.grad(o, (q, k, v), do))
    for a, b in zip(*out):
        assert a.shape == b.shape and a.stride() == b.stride() and torch.equal(a, b)


def test_hooks_on_saved_tensors_and_in_place_changes_are_seen(lib):
    from paper_2510_04212_amd.autograd import attention
    q, k, v = (t.requires_grad_(True) for t in _qkv(1, 2, 2, 64, 64, 64, "bhnd"))
    seen = []
    with torch.autograd.graph.saved_tensors_hooks(lambda t: seen.append(t.shape) or t.cpu(), lambda t: t.to(DEV)):
        o = attention(q, k, v)
    assert len(seen) == 5                                     # q, k, v, o, lse
    want = torch.autograd.grad(attention(q, k, v), q, torch.ones_like(o))[0]
    assert torch.equal(torch.autograd.grad(o, q, torch.ones_like(o))[0], want)
    o = attention(q, k, v)
    with torch.no_grad():
        v.zero_()
    with pytest.raises(RuntimeError, match="modified by an inplace operation"):
        torch.autograd.grad(o, q, torch.ones_like(o))


def test_what_was_refused_is_refused_the_same_way(lib):
    from paper_2510_04212_amd.autograd import attention
    q, k, v = _qkv(1, 2, 2, 64, 64, 64, "bhnd")
    with pytest.raises(ValueError):
        attention(q.float(), k, v)
    with pytest.raises(ValueError):
        attention(q, k, v[:, :1])
    for bad in (dict(variant=7), dict(softmax_scale=-1.0), dict(beta=0.5)):
        with pytest.raises(lib.AttnError):
            attention(q, k, v, **bad)
    with pytest.raises(lib.AttnError):
        attention(*_qkv(1, 2, 2, 64, 64, 80, "bhnd"))
    with pytest.raises(lib.AttnError):                        # a misaligned view
        flat = torch.zeros(64 * 64 + 8, dtype=torch.bfloat16, device=DEV)[4:4 + 64 * 64].view(1, 1, 64, 64)
        attention(flat, flat, flat)
    with pytest.raises(RuntimeError, match="setup_context"):  # function transforms: the Python node's own error
        torch.func.vmap(lambda a: attention(a, k, v))(q[None])
    with torch.autograd.forward_ad.dual_level(), pytest.raises(NotImplementedError, match="jvp"):
        attention(torch.autograd.forward_ad.make_dual(q, q), k, v)
    empty = torch.zeros((0, 2, 64, 64), dtype=torch.bfloat16, device=DEV)
    assert attention(empty, empty, empty).shape == empty.shape


@pytest.mark.parametrize("shape", [(1, 1, 1, 64), (1, 2, 1, 64), (2, 1, 2048, 64)], ids=str)
def test_expanded_dimensions_are_refused(lib, shape):
    """Rows (or heads, or a batch) that share storage: refused by both routes before any launch, also
    at the sizes where the forward takes a workspace."""
    from paper_2510_04212_amd.autograd import attention
    x = torch.zeros(shape, dtype=torch.bfloat16, device=DEV).expand(2, 2, 2048, 64)
    for call in (lambda: attention(x, x, x), lambda: lib.attn_fwd_strided(x, x, x, True, 0.125, 1)):
        with pytest.raises(lib.AttnError) as e:
            call()
        assert e.value.status == 2


@pytest.mark.parametrize("case", [CASES[0], CASES[2], CASES[3], CASES[5]], ids=str)     # every form of the node
def test_a_refused_gradient_is_refused_the_same_way(lib, case):
    """An incoming gradient that is not 16-byte aligned: AttnError with its status from both nodes."""
    from paper_2510_04212_amd import autograd as A
    data = _qkv(*case)
    for node in (lambda q, k, v: A.attention(q, k, v, True, 0.1, 1),
                 lambda q, k, v: A._FlashAttention.apply(q, k, v, True, 0.1, 1, None, None)):
        q, k, v = (t.detach().requires_grad_(True) for t in data)
        o = node(q, k, v)
        span = sum((n - 1) * s for n, s in zip(o.shape, o.stride())) + 1
        bad = torch.zeros(span + 4, dtype=torch.bfloat16, device=DEV)[4:].as_strided(o.shape, o.stride(), 4)
        assert bad.data_ptr() % 16 == 8
        for call in (lambda: torch.autograd.grad(o, q, bad, retain_graph=True), lambda: o.backward(bad, retain_graph=True)):
            with pytest.raises(lib.AttnError) as e:
                call()
            assert e.value.status == 2 and "misaligned" in str(e.value)
        good = torch.autograd.grad(o, (q, k, v), torch.ones_like(o))     # the graph is intact afterwards
        assert all(g.isfinite().all() for g in good)


CHANGES = {"host": lambda t: t.cpu(), "type": lambda t: t.double(), "shape": lambda t: t[:, :, :-1].contiguous(),
           "layout": lambda t: t.transpose(1, 2).contiguous().transpose(1, 2)}


@pytest.mark.parametrize("case", [CASES[0], CASES[2], CASES[3], CASES[5]], ids=str)     # every form of the node
@pytest.mark.parametrize("change", CHANGES)
def test_what_a_hook_hands_back_is_checked(lib, case, change):
    """K or O come back from a hook on saved tensors in host memory, or as another type, shape or layout than the
    kernels take: ValueError from both nodes, and nothing is launched."""
    from paper_2510_04212_amd import autograd as A
    data = _qkv(*case)
    for node in (lambda q, k, v: A.attention(q, k, v, True, 0.1, 1),
                 lambda q, k, v: A._FlashAttention.apply(q, k, v, True, 0.1, 1, None, None)):
        for which in (1, 3):                                  # of q, k, v, o, lse
            q, k, v = (t.detach().requires_grad_(True) for t in data)
            order = iter(range(5))
            unpack = lambda p: CHANGES[change](p[1]) if p[0] == which else p[1]
            with torch.autograd.graph.saved_tensors_hooks(lambda t: (next(order), t), unpack):
                o = node(q, k, v)
            with pytest.raises(ValueError):
                torch.autograd.grad(o, (q, k, v), torch.ones_like(o))
