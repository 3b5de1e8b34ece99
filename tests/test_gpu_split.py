"""GPU tests of the paths that share one block's work between wave groups or work-groups and add
partial results: sizes on both sides of the rules that choose them, remainders of tiles and blocks,
against the fp64 oracle (the tolerances are those of the other parity tests)."""
import pytest
import torch

from test_gpu_parity import DEV, check_head
from test_gpu_rect import _inputs, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [32, 64, 96, 128])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("Nq,Nk", [(511, 511), (512, 512), (545, 545), (640, 640), (33, 600), (700, 520)])
def test_dkdv_with_two_wave_groups(lib, Nq, Nk, d, causal):
    """From 512 keys on, few heads: two wave groups take alternate 32-query blocks (odd numbers of
    them, partial ones, a group that meets none at all) and add their dK, dV."""
    x = _inputs(3 * Nq + Nk + d, 1, 2, Nq, Nk, d, scale=1.25)
    got = _run(lib, x, causal, d ** -0.5, 1)
    for h in range(2):
        check_head(got, x, 0, h, causal, d ** -0.5, 1, label=f"groups {Nq}x{Nk} d{d} c{causal}")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N", [512, 577])
def test_grouped_queries_with_two_wave_groups(lib, N, d):
    """dK, dV of a shared head are the float32 sum over its query heads: per head the oracle-checked
    path on repeated K, V (same kernels, one head at a time), summed in float64."""
    B, H, Hkv = 1, 4, 2
    x = _inputs(N + d, B, H, N, N, d)
    K, V = x["K"][:, :Hkv].contiguous(), x["V"][:, :Hkv].contiguous()
    O, L = lib.attn_fwd_gqa(x["Q"], K, V, True, d ** -0.5, 1)
    dQ, dK, dV = lib.attn_bwd_gqa(x["Q"], K, V, O, x["dO"], L, True, d ** -0.5, 1)
    rep = lambda t: t.repeat_interleave(H // Hkv, 1).contiguous()
    _, dKx, dVx = lib.attn_bwd(x["Q"], rep(K), rep(V), O, x["dO"], L, True, d ** -0.5, 1)
    for got, per in ((dK, dKx), (dV, dVx)):
        want = per.double().view(B, Hkv, H // Hkv, N, d).sum(2)
        # each addend was rounded to bf16 (half an ulp, 2^-9 of its size), so was the result
        assert ((got.double() - want).norm() / want.norm()).item() <= 2.0 ** -8
