"""Rows of the forward that meet in one instruction stay apart: a query row that is not finite (the row sums of some
kernels are taken for pairs of rows, r and r ^ 16, in one matrix instruction) leaves every other row as it was."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", [0, 1, 2])
@pytest.mark.parametrize("d,causal", [(32, True), (64, True), (64, False), (96, True), (96, False), (128, True), (128, False), (256, True)])
@pytest.mark.parametrize("N", [70, 256])
def test_a_row_that_is_not_finite_stays_alone(lib, variant, d, causal, N):
    g = torch.Generator(device="cuda:0").manual_seed(d + N)
    q, k, v = (torch.randn((1, 2, N, d), generator=g, device="cuda:0").to(torch.bfloat16) for _ in range(3))
    alpha = d ** -0.5
    ref, ref_l = lib.attn_fwd(q, k, v, causal, alpha, variant)
    hurt = [3, 21, 64, N - 1]
    qn = q.clone()
    qn[:, :, hurt[:2], 0] = float("nan")
    qn[:, :, hurt[2:], 0] = float("inf")       # scores +-inf: NaN where they meet, as in the formula
    for extras in (False, True):
        if extras:
            f = lib.attn_fwd_opt(qn, k, v, causal, alpha, variant, want_O_hp=True)
            o, l = f["O"], f["LSE"]
        else:
            o, l = lib.attn_fwd(qn, k, v, causal, alpha, variant)
        torch.cuda.synchronize()
        assert not torch.isfinite(l[:, :, hurt]).any()
        others = [r for r in range(N) if r not in hurt]
        # the sums of the other rows of a wave may be taken in another order: one float32 step in l, so at most
        # one bf16 step in O (2^-7 of the value, and nothing where the value is exact)
        a, b = o[:, :, others].float(), ref[:, :, others].float()
        assert torch.isfinite(a).all() and ((a - b).abs() <= 2.0 ** -7 * b.abs()).all()
        assert (l[:, :, others] - ref_l[:, :, others]).abs().max() <= 1e-5 * (1 + ref_l.abs().max())


@pytest.mark.parametrize("variant", [0, 1, 2])
@pytest.mark.parametrize("d", [32, 64, 96, 128, 256])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("N", [70, 256, 1030])
def test_a_nan_row_is_nan_whatever_kernel_serves_it(lib, variant, d, causal, N):
    """Every score of the row is NaN, so l, O and LSE are: in the aligned, the bounds-checking and (N = 1030) the
    shared-out kernels, with and without optional outputs.  A row of zeros is for queries that see no key at all."""
    g = torch.Generator(device="cuda:0").manual_seed(d + N)
    q, k, v = (torch.randn((1, 2, N, d), generator=g, device="cuda:0").to(torch.bfloat16) for _ in range(3))
    hurt = [0, 3, 64, N - 1]
    q[:, :, hurt] = float("nan")
    others = [r for r in range(N) if r not in hurt]
    alpha = d ** -0.5
    runs = {"plain": dict(zip(("O", "LSE"), lib.attn_fwd(q, k, v, causal, alpha, variant)))}
    for option in (None, "single_rounding", "pv_e4m3", "guard_underflow"):
        runs[option] = lib.attn_fwd_opt(q, k, v, causal, alpha, variant, want_O_hp=True, want_counts=True,
                                        **({option: True} if option else {}))
    for name, f in runs.items():
        for t in ("O", "O_hp", "LSE"):
            if t in f:
                assert f[t][:, :, hurt].isnan().all(), (name, t)
                assert f[t][:, :, others].isfinite().all(), (name, t)
