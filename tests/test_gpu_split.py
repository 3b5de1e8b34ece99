"""GPU tests of the paths that share one block's work between wave groups or work-groups and add
partial results: sizes on both sides of the rules that choose them, remainders of tiles and blocks,
against the fp64 oracle (the tolerances are those of the other parity tests)."""
import numpy as np
import pytest
import torch

from oracle import exact, metrics
from test_gpu_parity import DEV, TOL_ABS, TOL_REL, check_head
from test_gpu_rect import _inputs, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [32, 64, 96, 128, 256])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("Nq,Nk", [(511, 511), (512, 512), (545, 545), (640, 640), (33, 600), (700, 520), (1, 513)])
def test_backward_with_wave_groups(lib, Nq, Nk, d, causal):
    """From 512 keys on, two heads: blocks of 32 rows whose eight wave groups (d = 96, 128: four; dK/dV at d = 64 under the mask: two on
    64 keys) take alternate 32-query blocks (dK/dV) or 32-key blocks (dQ) - numbers of them no group count divides, partial
    ones, groups that meet none at all - and add their sums."""
    x = _inputs(3 * Nq + Nk + d, 1, 2, Nq, Nk, d, scale=1.25)
    got = _run(lib, x, causal, d ** -0.5, 1)
    for h in range(2):
        check_head(got, x, 0, h, causal, d ** -0.5, 1, label=f"groups {Nq}x{Nk} d{d} c{causal}")


# heads, queries, keys, d, mask -> the forms of dQ and dK/dV (csrc/bwd_forms.hpp; 6: two groups on 64 keys)
RECTANGLES = [
    (16, 577, 700, 64, True, 4, 4), (16, 700, 577, 64, True, 4, 4), (17, 640, 1000, 32, True, 4, 4), (16, 1000, 1025, 96, True, 4, 4),
    (16, 1100, 1101, 128, True, 4, 4), (14, 700, 640, 64, False, 4, 4), (15, 600, 1000, 96, False, 4, 4), (21, 500, 600, 32, False, 4, 4),
    (32, 577, 700, 64, True, 2, 6), (40, 640, 520, 32, True, 2, 6), (33, 530, 600, 96, True, 2, 6), (48, 700, 900, 64, True, 2, 6),
    (24, 500, 600, 128, True, 2, 4), (18, 700, 530, 128, False, 2, 4), (24, 300, 700, 128, True, 2, 4),
    (64, 560, 600, 64, False, 2, 6), (60, 600, 513, 32, False, 2, 6), (52, 575, 570, 96, False, 2, 6), (40, 130, 1024, 96, False, 4, 6)]


@pytest.mark.parametrize("H,Nq,Nk,d,causal,dq,dkdv", RECTANGLES, ids=str)
def test_four_and_two_wave_groups_on_rectangles(lib, H, Nq, Nk, d, causal, dq, dkdv):
    """Between 65 and 384 blocks: four groups and two on 64 rows, with more keys than queries and fewer (a mask that is shifted
    either way, queries that see no key), against the oracle."""
    x = _inputs(H + 3 * Nq + Nk + d, 1, H, Nq, Nk, d, scale=1.25)
    got = _run(lib, x, causal, d ** -0.5, 1)
    for h in (0, H - 1):
        check_head(got, x, 0, h, causal, d ** -0.5, 1, label=f"rectangle H{H} {Nq}x{Nk} d{d} c{causal}")


@pytest.mark.parametrize("d", [32, 64, 96, 128])
@pytest.mark.parametrize("H,N,causal", [(33, 1024, True), (40, 897, True), (17, 1024, False), (20, 1000, False)])
def test_dkdv_with_two_wave_groups(lib, H, N, d, causal):
    """More blocks than the four-group rule takes (256 with, 128 without a mask): two groups on 128 keys, or, up to one and a half
    blocks per CU under the mask, two on 64 at d < 128 (33 heads, which run in pairs: one at d < 96)."""
    x = _inputs(H + N + d, 1, H, N, N, d, scale=1.25)
    got = _run(lib, x, causal, d ** -0.5, 1)
    for h in (0, H - 1):
        check_head(got, x, 0, h, causal, d ** -0.5, 1, label=f"two groups H{H} N{N} d{d} c{causal}")


@pytest.mark.parametrize("d", [32, 64])
@pytest.mark.parametrize("H,N,causal", [(264, 200, True), (520, 65, True), (72, 1000, True), (513, 128, False), (260, 161, False),
                                        (515, 300, True), (342, 384, True), (341, 384, True)])
def test_dkdv_with_three_waves_per_simd(lib, H, N, d, causal):
    """More than two 128-key blocks per CU: aligned, ragged, shorter than a block.  Head counts that are not in eights run as
    mirrored pairs of blocks and take it from more than four blocks per CU on (342 heads of three; 341 are one too few)."""
    x = _inputs(H + N + d, 1, H, N, N, d, scale=1.25)
    got = _run(lib, x, causal, d ** -0.5, 1)
    for h in (0, H // 2, H - 1):
        check_head(got, x, 0, h, causal, d ** -0.5, 1, label=f"three waves H{H} N{N} d{d} c{causal}")


@pytest.mark.parametrize("d", [64, 96, 128, 256])
@pytest.mark.parametrize("H,N", [(512, 400), (513, 384), (512, 385)])
def test_causal_forward_and_dq_in_mirrored_pairs(lib, H, N, d):
    """From 1024 pairs of query blocks on a work-group takes two blocks one after the other: ragged lengths, an odd number
    of blocks (the middle one has no partner), a last block of one row.  (From d = 96 on the forward's pipeline starts anew.)"""
    x = _inputs(H + N + d, 1, H, N, N, d, scale=1.25)
    for variant in (0, 1):
        got = _run(lib, x, True, d ** -0.5, variant)
        for h in (0, H // 2, H - 1):
            check_head(got, x, 0, h, True, d ** -0.5, variant, label=f"pairs H{H} N{N} d{d} v{variant}")


@pytest.mark.parametrize("H,N,causal", [(130, 520, True), (104, 640, True), (70, 600, False), (66, 512, False), (300, 97, True)])
def test_dkdv_with_one_wave_group_at_128(lib, H, N, causal):
    """More key blocks than the wave groups take (512 with, 256 without a mask), or short sequences: one group, V_j in LDS."""
    x = _inputs(H + N, 1, H, N, N, 128, scale=1.25)
    got = _run(lib, x, causal, 128 ** -0.5, 1)
    for h in (0, H - 1):
        check_head(got, x, 0, h, causal, 128 ** -0.5, 1, label=f"one group H{H} N{N} c{causal}")


@pytest.mark.parametrize("H,N", [(16, 1500), (16, 1536), (8, 3970), (16, 2048), (16, 1499), (17, 1500), (16, 2049)])
def test_dq_at_256_with_two_wave_groups(lib, H, N):
    """Causal, 129 to 256 query blocks, head counts in eights, from 1500 keys on: two groups on 64 queries; one beside that."""
    x = _inputs(H + N, 1, H, N, N, 256, scale=1.25)
    got = _run(lib, x, True, 1.0 / 16, 1)
    check_head(got, x, 0, H - 1, True, 1.0 / 16, 1, label=f"two groups H{H} N{N}")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N", [512, 577])
def test_grouped_queries_with_wave_groups(lib, N, d):
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


@pytest.mark.parametrize("d", [32, 64, 96, 128, 256])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("Nq,Nk", [(1, 1024), (33, 1090), (64, 4097), (1024, 1024), (1100, 1500), (1500, 1030)])
def test_forward_shared_out_over_key_tiles(lib, Nq, Nk, d, causal):
    """Few query blocks and at least 1024 keys: shares of a block's key tiles, some of them without a
    visible key, partial last tiles and blocks, rows that see no key at all."""
    assert lib.raw().attn_fwd_workspace_bytes(1, 2, Nq, Nk, d, int(causal), 1) > 0
    x = _inputs(5 * Nq + Nk + d, 1, 2, Nq, Nk, d, scale=1.25)
    for variant in (0, 1):
        got = _run(lib, x, causal, d ** -0.5, variant)
        for h in range(2):
            check_head(got, x, 0, h, causal, d ** -0.5, variant, label=f"shares {Nq}x{Nk} d{d} c{causal} v{variant}")


def test_forward_shared_out_takes_strides_and_grouped_heads(lib):
    """The same shares whatever the layout: strided views and grouped heads give the bits of the
    contiguous call on repeated heads; a workspace that is too small is refused."""
    B, H, Hkv, N, d = 1, 4, 2, 1200, 64
    x = _inputs(9, B, H, N, N, d)
    rep = lambda t: t[:, :Hkv].repeat_interleave(H // Hkv, 1).contiguous()
    K, V = rep(x["K"]), rep(x["V"])
    O, L = lib.attn_fwd(x["Q"], K, V, True, 0.125, 1)
    Og, Lg = lib.attn_fwd_gqa(x["Q"], x["K"][:, :Hkv].contiguous(), x["V"][:, :Hkv].contiguous(), True, 0.125, 1)
    s = lambda t: t.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)
    Os, Ls = lib.attn_fwd_strided(s(x["Q"]), s(K), s(V), True, 0.125, 1)
    for o, l in ((Og, Lg), (Os, Ls)):
        assert torch.equal(o, O) and torch.equal(l, L)
    p = lambda t: t.data_ptr()
    ws = torch.empty(1 << 20, dtype=torch.uint8, device=DEV)
    assert lib.raw().attn_fwd_ws(p(x["Q"]), p(K), p(V), p(O), p(L), p(ws), 256, 0, 0, 0, B, H, H, N, N, d, 1,
                                 0.125, 1, 2.0, 1e-3, None) == 4


@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("H,Nq,Nk,d,causal", [(2, 1024, 1024, 64, True), (2, 64, 4097, 128, True), (3, 1, 1500, 96, False),
                                              (1, 2100, 2100, 32, True), (8, 2048, 2048, 256, False),
                                              (48, 130, 2560, 64, True), (43, 200, 2600, 128, False)])
def test_shares_round_the_probabilities_of_the_one_pass_kernel(lib, H, Nq, Nk, d, causal, variant):
    """Every share starts from the normaliser a single pass would have reached, so P-bar is rounded the same
    and only float32 sums change their order.  T tiles in another order differ by about sqrt(T) 2^-24
    sum|terms| / |sum| <= 2e-5; an element takes another bf16 value (2^-8 off at most) when that crosses a
    boundary of one of its two roundings: 4 x 2e-5 / 2^-8 = 2e-2 of them at most, sqrt(2e-2) 2^-8 = 6e-4 in the
    2-norm (P-bar rounded against the share's own maximum: 1e-3 to 3e-3).  Seen: 2e-5 .. 4e-5, and 3.8e-4 where
    Alg. 1 adds two unit probabilities, whose sums lie on those boundaries.
    Repeated keys in the first tile make Alg. 3 move the normaliser there: it has to stay moved in
    all later shares."""
    x = _inputs(11 * H + Nq + Nk + d, 1, H, Nq, Nk, d, scale=1.5)
    x["K"][:, :, 1:16:2] = x["K"][:, :, 0:16:2]
    x["Q"][:, :, ::2] = x["K"][:, :, 3:4] + 0.5 * x["Q"][:, :, ::2]
    assert lib.raw().attn_fwd_workspace_bytes(1, H, Nq, Nk, d, int(causal), variant) > 0
    if Nq == Nk:
        O, L = lib.attn_fwd(x["Q"], x["K"], x["V"], causal, d ** -0.5, variant)
        ref = lib.attn_fwd_opt(x["Q"], x["K"], x["V"], causal, d ** -0.5, variant, want_counts=True)
        O1, L1 = ref["O"], ref["LSE"]
        assert variant == 0 or ref["fired"].sum() > 0
    else:
        O, L = lib.attn_fwd_rect(x["Q"], x["K"], x["V"], causal, d ** -0.5, variant)
        O1, L1 = torch.empty_like(O), torch.empty_like(L)
        p = lambda t: t.data_ptr()
        assert lib.raw().attn_fwd_rect(p(x["Q"]), p(x["K"]), p(x["V"]), p(O1), p(L1), 1, H, Nq, Nk, d, int(causal), d ** -0.5,
                                       variant, 2.0, 1e-3, torch.cuda.current_stream().cuda_stream) == 0
    differ = (O != O1).double().mean().item()
    rel = ((O.double() - O1.double()).norm() / O1.double().norm()).item()
    print(f"shares H{H} {Nq}x{Nk} d{d} c{causal} v{variant}: differ {differ:.1e} rel {rel:.1e}")
    assert differ <= 2e-2 and rel <= 6e-4
    assert torch.allclose(L, L1, rtol=0, atol=2e-6 * L1.abs().max().item())


@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("N", [1024, 1030])
def test_shares_with_infinite_scores(lib, N, variant):
    """Rows whose scores overflow to -inf, to +inf, or in some tiles only, give what the one-pass kernel
    gives (NaN or 0, by the instantiation that serves the size)."""
    x = _inputs(N, 1, 2, N, N, 64)
    x["Q"][:, :, 5] = 3e38
    x["Q"][:, :, 700] = -3e38
    x["Q"][:, :, 900] = 3e38
    x["K"][:, 0] = -x["K"][:, 0].abs()
    x["K"][:, 1, :640] = -x["K"][:, 1, :640].abs()
    x["K"][:, 1, 640:] = 0
    O, L = lib.attn_fwd(x["Q"], x["K"], x["V"], True, 0.125, variant)
    ref_O, ref_L = torch.empty_like(O), torch.empty_like(L)
    p = lambda t: t.data_ptr()
    assert lib.raw().attn_fwd_workspace_bytes(1, 2, N, N, 64, 1, variant) > 0
    assert lib.raw().attn_fwd_ex(p(x["Q"]), p(x["K"]), p(x["V"]), p(ref_O), p(ref_L), 1, 2, N, 64, 1, 0.125, variant,
                                 2.0, 1e-3, torch.cuda.current_stream().cuda_stream) == 0
    for a, b in ((O, ref_O), (L, ref_L)):
        assert torch.equal(a.isnan(), b.isnan())
        ok = ~b.isnan()
        assert torch.allclose(a[ok].float(), b[ok].float(), rtol=2.0 ** -7, atol=1e-4)
    assert ref_O[0, 0, 5].isnan().all().item() == (N % 128 == 0)


@pytest.mark.parametrize("N,stride,d", [(200, (1 << 24) - 8, 128), (512, 9_000_000, 128), (512, 8_388_616, 64), (600, (1 << 24) - 8, 64),
                                        (700, 9_000_000, 32)])
def test_rows_far_apart(lib, N, stride, d):
    """Row strides at which the last rows of a 128-row tile lie 2 to 4 GiB behind its first (V_j at d = 128, and the 128-row
    tiles of wave groups), and those of a 256-row tile (eight groups at d <= 64) up to 8 GiB: the bits of the contiguous call."""
    x = _inputs(N, 1, 1, N, N, d)
    far = torch.empty((N - 1) * stride + 8 * d, dtype=torch.bfloat16, device=DEV)
    view = lambda i: far[i * d:].as_strided((1, 1, N, d), (8, 8, stride, 1))
    t = {n: view(i) for i, n in enumerate(("Q", "K", "V", "dO", "O", "dQ", "dK", "dV"))}
    for n in ("Q", "K", "V", "dO"):
        t[n].copy_(x[n])
    want = _run(lib, x, True, d ** -0.5, 1)
    _, L = lib.attn_fwd_strided(t["Q"], t["K"], t["V"], True, d ** -0.5, 1, O=t["O"])
    lib.attn_bwd_strided(t["Q"], t["K"], t["V"], t["O"], t["dO"], L, True, d ** -0.5, 1, dQ=t["dQ"], dK=t["dK"], dV=t["dV"])
    assert torch.equal(L, want["L"])
    for n in ("O", "dQ", "dK", "dV"):
        assert torch.equal(t[n], want[n]), n


def test_the_caller_decides_about_the_workspace(lib):
    """Few heads, 1200 keys.  Own outputs: nothing is allocated and one pass runs, as the C entry points
    without a workspace do; own workspace: used, or refused when it is too small or misaligned; one_pass: the bits
    of attn_fwd_opt.  In every layout."""
    B, H, N, d = 1, 4, 1200, 64
    x = _inputs(9, B, H, N, N, d)
    args = (x["Q"], x["K"], x["V"], True, 0.125, 1)
    need = lib.fwd_workspace_bytes(B, H, N, N, d, True, 1)
    assert need > 0
    ws = torch.empty(need + 256, dtype=torch.uint8, device=DEV)
    O, L = lib.attn_fwd(*args)
    one = lib.attn_fwd_opt(*args)
    s = lambda t: t.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)
    st = (s(x["Q"]), s(x["K"]), s(x["V"]), True, 0.125, 1)
    forms = {"plain": (lib.attn_fwd, args), "strided": (lib.attn_fwd_strided, st), "gqa": (lib.attn_fwd_gqa, args),
             "rect": (lib.attn_fwd_rect, args)}
    for name, (f, a) in forms.items():
        o, l = f(*a, one_pass=True)
        assert torch.equal(o, one["O"]) and torch.equal(l, one["LSE"]), name
        o, l = f(*a, workspace=ws[:need])
        assert torch.equal(o, O) and torch.equal(l, L), name
        for bad in (ws[:need - 16], ws[8:]):
            with pytest.raises(lib.AttnError) as e:
                f(*a, workspace=bad)
            assert e.value.status == 4, name
        if name in ("plain", "strided"):
            o, l = torch.empty_like(a[0]), torch.empty_like(L)
            count = lambda: torch.cuda.memory_stats()["allocation.all.allocated"]
            before = count()
            f(*a, O=o, LSE=l)
            f(*a, O=o, LSE=l, workspace=ws)
            assert count() == before, name
            f(*a, O=o, LSE=l)
            assert torch.equal(o, one["O"]) and torch.equal(l, one["LSE"]), name
    with pytest.raises(ValueError):
        lib.attn_fwd(*args, workspace=torch.empty(need, dtype=torch.uint8))
    p = lambda t: t.data_ptr()
    o, l = torch.empty_like(O), torch.empty_like(L)
    assert lib.raw().attn_fwd_ws(p(x["Q"]), p(x["K"]), p(x["V"]), p(o), p(l), None, 0, 0, 0, 0, B, H, H, N, N, d, 1, 0.125, 1,
                                 2.0, 1e-3, torch.cuda.current_stream().cuda_stream) == 0
    assert torch.equal(o, one["O"]) and torch.equal(l, one["LSE"])


@pytest.mark.parametrize("layout", ["bnhd", "fused"])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("H,N,d", [(2, 512, 32), (2, 512, 64), (3, 700, 64), (2, 640, 96), (2, 512, 128), (3, 1025, 128),
                                   (2, 512, 256), (2, 600, 256), (33, 1024, 96), (33, 1024, 128), (17, 1000, 128),
                                   (72, 512, 64), (72, 513, 32), (40, 600, 64), (40, 600, 96), (52, 570, 96), (16, 577, 64),
                                   (16, 700, 96), (24, 600, 128)], ids=str)
def test_strides_with_wave_groups(lib, H, N, d, causal, layout):
    """The wave-group kernels (blocks of 32 rows, four groups, two on 64 and on 128 rows, dQ's two at d = 256) on strided tensors: the
    bits of the contiguous call, which the oracle tests cover."""
    x = _inputs(H + N + d, 1, H, N, N, d, scale=1.25)
    O, L = lib.attn_fwd(x["Q"], x["K"], x["V"], causal, d ** -0.5, 1)
    want = lib.attn_bwd(x["Q"], x["K"], x["V"], O, x["dO"], L, causal, d ** -0.5, 1)
    if layout == "fused":       # every bf16 tensor a slice of one [1, N, 5, H, d] buffer (outputs: of another)
        buf, out = (torch.full((1, N, 5, H, d), float("nan"), dtype=torch.bfloat16, device=DEV) for _ in range(2))
        part = lambda t, i: t[:, :, i].permute(0, 2, 1, 3)
    else:
        buf, out = (torch.full((5, 1, N, H, d), float("nan"), dtype=torch.bfloat16, device=DEV) for _ in range(2))
        part = lambda t, i: t[i].permute(0, 2, 1, 3)
    q, k, v, do, o = (part(buf, i) for i in range(5))
    for t, src in ((q, "Q"), (k, "K"), (v, "V"), (do, "dO")):
        t.copy_(x[src])
    assert q.stride(2) != d
    _, Ls = lib.attn_fwd_strided(q, k, v, causal, d ** -0.5, 1, O=o)
    got = lib.attn_bwd_strided(q, k, v, o, do, Ls, causal, d ** -0.5, 1, *(part(out, i) for i in range(3)))
    assert torch.equal(o, O) and torch.equal(Ls, L)
    for n, a, b in zip(("dQ", "dK", "dV"), got, want):
        assert torch.equal(a, b), n
    for i in (3, 4):            # nothing is written beside the outputs
        assert part(out, i).isnan().all()


@pytest.mark.parametrize("Hkv,group,N,d,causal", [
    (2, 2, 512, 32, False), (2, 2, 512, 32, True), (2, 4, 577, 64, False), (2, 2, 545, 96, True), (2, 2, 512, 96, False),
    (1, 4, 700, 128, False), (2, 2, 640, 128, True),                                  # dK/dV: blocks of 32 keys
    (16, 2, 577, 32, True), (16, 2, 577, 64, True), (16, 2, 640, 128, True), (27, 2, 600, 96, True), (34, 2, 512, 64, True),
    (16, 2, 600, 128, False), (16, 4, 520, 64, False), (20, 2, 640, 96, False),       # four groups (65 to 256 key blocks, 128 without a mask)
    (52, 2, 640, 96, True), (52, 2, 640, 128, True), (65, 2, 500 + 12, 128, True),    # two groups (257 to 512 key blocks)
    (27, 2, 640, 32, False), (27, 2, 640, 64, False), (27, 3, 600, 96, False), (33, 2, 512, 128, False),   # two (129 to 256)
    (52, 2, 640, 64, True), (52, 2, 640, 64, False), (2, 2, 640, 256, False)], ids=str)                        # one
def test_grouped_queries_with_wave_groups_against_the_oracle(lib, Hkv, group, N, d, causal):
    """dQ per query head, dK and dV of a shared head the sum over its query heads, all in 64 bits."""
    H = Hkv * group
    x = _inputs(H + N + d, 1, H, N, N, d, scale=1.25)
    x["K"], x["V"] = x["K"][:, :Hkv].contiguous(), x["V"][:, :Hkv].contiguous()
    x["dO"] = x["dO"] / group                      # sums stay in the range the tolerances are for
    O, L = lib.attn_fwd_gqa(x["Q"], x["K"], x["V"], causal, d ** -0.5, 1)
    dQ, dK, dV = lib.attn_bwd_gqa(x["Q"], x["K"], x["V"], O, x["dO"], L, causal, d ** -0.5, 1)
    f64 = lambda t, h: t[0, h].double().cpu().numpy()
    for hk in sorted({0, Hkv - 1}):
        sums = [0.0, 0.0]
        for h in range(hk * group, (hk + 1) * group):
            ref = exact.forward_backward(f64(x["Q"], h), f64(x["K"], hk), f64(x["V"], hk), f64(x["dO"], h), d ** -0.5, causal)
            for n, got, want in (("O", O, ref[0]), ("dQ", dQ, ref[2])):
                assert metrics.max_abs(f64(got, h), want) <= TOL_ABS and metrics.rel_l2(f64(got, h), want) <= TOL_REL, (n, h)
            sums = [a + b for a, b in zip(sums, ref[3:5])]
        for n, got, want in (("dK", dK, sums[0]), ("dV", dV, sums[1])):
            g = f64(got, hk)
            assert np.isfinite(g).all() and metrics.max_abs(g, want) <= TOL_ABS and metrics.rel_l2(g, want) <= TOL_REL, (n, hk)
