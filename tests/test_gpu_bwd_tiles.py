"""GPU test of the two backward kernels where their tiles end: sequence lengths around 16, 32, 64 and 128 rows, at every head
size, on grids that take one, two, four and eight wave groups and the kernels with three waves per SIMD.

The kernels get LSE and delta rounded from float64, so every entry has a bound of its own: P and dS are rounded to bf16 once
as operands and the result once when stored (each 2^-8 relative), and the float32 sums behind S, dP and the exponent add
less than 2^-12 of the absolute values that enter them.  A row or column in the wrong place is off by its own size.
"""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
U, SLACK = 2.0 ** -8, 2.0 ** -12


def _check(lib, B, H, N, d, causal):
    g = torch.Generator(device=DEV).manual_seed(N + d)
    q, k, v, do = (torch.randn((B, H, N, d), generator=g, device=DEV).to(torch.bfloat16) for _ in range(4))
    alpha = 1.0 / math.sqrt(d)
    Q, K, V, G = (t.double() for t in (q, k, v, do))
    S = alpha * (Q @ K.transpose(-1, -2))
    if causal:
        S = S.masked_fill(torch.ones((N, N), dtype=torch.bool, device=DEV).triu(1), -math.inf)
    L = torch.logsumexp(S, -1)
    P = torch.exp(S - L[..., None])
    dP = G @ V.transpose(-1, -2)
    delta = (P * dP).sum(-1)
    dS = P * (dP - delta[..., None])
    inner = P * (G.abs() @ V.abs().transpose(-1, -2) + delta.abs()[..., None])       # what the float32 sums of dS run over
    t = lambda x: x.transpose(-1, -2)
    want = {"dQ": alpha * (dS @ K), "dK": alpha * (t(dS) @ Q), "dV": t(P) @ G}
    part = {"dQ": alpha * ((U * dS.abs() + SLACK * inner) @ K.abs()), "dK": alpha * (t(U * dS.abs() + SLACK * inner) @ Q.abs()),
            "dV": (U + SLACK) * (t(P) @ G.abs())}
    dK, dV = lib.attn_bwd_dkdv(q, k, v, do, L.float(), delta.float(), causal, alpha)
    dQ = lib.attn_bwd_dq(q, k, v, do, L.float(), delta.float(), causal, alpha)
    torch.cuda.synchronize()
    for name, got in (("dQ", dQ), ("dK", dK), ("dV", dV)):
        bound = part[name] + U * (want[name].abs() + part[name]) + 1e-30
        over = (got.double() - want[name]).abs() / bound
        assert not got.isnan().any() and float(over.max()) <= 1.0, (name, float(over.max()))


@pytest.mark.parametrize("B,H,N,d,causal", [
    # blocks of 32 rows (eight wave groups at d <= 64, four beyond), grids up to and just above a work-group per CU
    (1, 1, 512, 64, True), (1, 1, 513, 64, True), (1, 3, 640, 32, True), (2, 4, 1000, 64, False), (1, 8, 1024, 64, True),
    (2, 8, 1024, 64, True), (1, 12, 1024, 64, True), (1, 13, 1025, 32, False),
    (1, 1, 512, 128, True), (1, 2, 700, 128, True), (1, 3, 1000, 96, False), (1, 8, 1024, 128, True), (2, 4, 640, 128, False),
    # dQ and dK/dV at d <= 64 with two wave groups on 64 rows: just above one block of 128 per CU, at the rule's upper limits, one block beyond
    (5, 13, 512, 64, True), (4, 13, 513, 64, True), (8, 12, 512, 64, False), (1, 97, 512, 64, True), (1, 33, 1000, 32, False),
    (8, 16, 512, 32, True), (1, 129, 512, 32, True),
    # the same at every head size, below one block per CU (short and longer sequences under the mask) and above
    (1, 33, 513, 64, True), (1, 33, 512, 32, True), (3, 8, 1025, 64, True), (1, 25, 1100, 96, True), (1, 33, 513, 96, True), (8, 12, 512, 96, False),
    (5, 13, 513, 96, True), (1, 17, 512, 128, True), (2, 33, 513, 128, True), (1, 80, 512, 128, True), (1, 17, 513, 128, False), (4, 8, 512, 128, False),
    # at and beyond the lines that leave two groups for one or four: short sequences at d = 128, grids that do not divide over the XCDs, keys in the
    # thousands, dK/dV at d = 64 in pairs of blocks
    (1, 53, 768, 128, True), (1, 64, 512, 128, True), (1, 20, 1100, 128, True), (1, 58, 640, 96, False), (1, 64, 640, 96, False), (1, 54, 576, 96, False),
    (1, 3, 3000, 128, False), (1, 5, 2048, 128, False), (1, 22, 640, 64, True), (1, 11, 768, 64, True), (1, 24, 768, 32, True), (1, 23, 1024, 32, True)])
def test_every_entry_on_small_grids_of_longer_sequences(lib, B, H, N, d, causal):
    _check(lib, B, H, N, d, causal)


@pytest.mark.parametrize("N", [1, 15, 17, 33, 64, 65, 127, 128, 256, 320])
@pytest.mark.parametrize("B,H,d,causal", [
    (1, 1, 32, True), (1, 2, 64, False), (1, 2, 64, True), (2, 1, 96, True), (1, 2, 128, True), (1, 1, 128, False), (1, 1, 256, True),
    (9, 15, 64, True), (9, 15, 128, True), (9, 15, 256, False), (24, 32, 64, True), (24, 32, 64, False), (24, 32, 32, True), (8, 32, 128, True)])
def test_every_entry_at_the_edges_of_the_tiles(lib, N, B, H, d, causal):
    _check(lib, B, H, N, d, causal)
