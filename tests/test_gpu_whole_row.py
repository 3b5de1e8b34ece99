"""GPU test of the whole-row form of Alg. 3 where its two passes over the key tiles meet: no tile, one, odd and even numbers
of tiles, partial ones, more keys than queries and fewer (rows that see no key).

The output is compared entry by entry with float64.  P-bar and the unnormalised output are rounded to bf16 once, the quotient
once, and the row sum is of the rounded P-bar (each 2^-8 relative); float32 sums and the exponent add less than 2^-12.
"""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
U, SLACK = 2.0 ** -8, 2.0 ** -12


@pytest.mark.parametrize("Nq,Nk", [(1, 1), (1, 64), (33, 65), (128, 128), (129, 129), (64, 192), (300, 256), (256, 100), (320, 320), (5, 700)])
@pytest.mark.parametrize("d,causal", [(32, True), (64, True), (64, False), (96, True), (128, True), (128, False), (256, True)])
def test_both_passes_see_every_tile(lib, Nq, Nk, d, causal):
    g = torch.Generator(device=DEV).manual_seed(Nq + Nk + d)
    q, k, v = (torch.randn((2, 3, n, d), generator=g, device=DEV).to(torch.bfloat16) for n in (Nq, Nk, Nk))
    k[:, :, Nk // 2] = k[:, :, 0]             # a tie across the tiles, the largest score of some rows
    alpha = 1.0 / math.sqrt(d)
    S = alpha * (q.double() @ k.double().transpose(-1, -2))
    seen = torch.ones((Nq, Nk), dtype=torch.bool, device=DEV)
    if causal:
        seen = seen.tril(Nk - Nq)
    S = S.masked_fill(~seen, -math.inf)
    some = seen.any(-1)
    L = torch.logsumexp(S, -1)
    P = torch.where(some[:, None], torch.exp(S - torch.where(some, L, 0.0)[..., None]), 0.0)
    want, part = P @ v.double(), P @ v.double().abs()
    O, LSE = lib.attn_fwd_rect(q, k, v, causal, alpha, lib.MITIGATED_ROW)
    torch.cuda.synchronize()
    bound = (2 * U + SLACK) * part + 2 * U * (want.abs() + part * 2 * U) + 1e-30
    assert not O.isnan().any()
    over = (O.double() - want).abs() / bound
    assert float(over.max()) <= 1.0, float(over.max())
    assert torch.equal(torch.isneginf(LSE), ~some.expand_as(LSE))
    assert float((LSE.double() - L)[:, :, some].abs().max()) <= U + SLACK * 8


@pytest.mark.parametrize("N", [1, 63, 64, 65, 128, 200, 320, 449])
@pytest.mark.parametrize("d,causal", [(32, True), (64, True), (64, False), (96, True), (128, False), (256, True)])
def test_the_rule_fires_on_whole_rows(lib, N, d, causal):
    """Which rows the rule moved, against the two largest scores of the whole row in float64.  Repeated keys, in one tile and
    tiles apart, and queries close to them.  A score's float32 sum is off by at most d 2^-24 of the sum of its products'
    magnitudes: a row whose gap (two scores) lies that close to eps may go either way, unless its two largest scores belong to
    equal keys, whose scores are equal bit for bit."""
    g = torch.Generator(device=DEV).manual_seed(N + d)
    q, k, v = (torch.randn((2, 3, N, d), generator=g, device=DEV).to(torch.bfloat16) for _ in range(3))
    k[:, :, N // 2] = k[:, :, 0]              # a tie across the tiles
    k[:, :, N - 1] = k[:, :, N // 3]
    q[:, :, ::2] += k[:, :, N // 2].unsqueeze(2)
    q[:, :, 1::2] -= k[:, :, N // 3].unsqueeze(2)
    alpha, eps = 1.0 / math.sqrt(d), 1e-3
    Q, K = q.double(), k.double()
    seen = torch.ones((N, N), dtype=torch.bool, device=DEV)
    if causal:
        seen = seen.tril()
    S = (alpha * (Q @ K.transpose(-1, -2))).masked_fill(~seen, -math.inf)
    top = S.topk(min(2, N), -1).values
    gap = top[..., 0] - top[..., -1] if N > 1 else torch.full_like(top[..., 0], math.inf)
    slack = 2 * d * 2.0 ** -24 * alpha * (Q.abs() @ K.abs().transpose(-1, -2)).amax(-1)
    got = lib.attn_fwd_opt(q, k, v, causal, alpha, lib.MITIGATED_ROW, eps=eps, want_counts=True)["fired"]
    sure = (((gap - eps).abs() > slack) | (gap < 1e-12)) & (top[..., 0].abs() > slack)
    assert torch.equal(got[sure] != 0, (gap <= eps)[sure])
    assert sure.double().mean() > 0.9
    if N >= 64:
        assert (got != 0).any() and (got == 0).any()
