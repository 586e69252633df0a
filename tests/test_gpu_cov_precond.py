"""GPU parity of the covariance (Eq. (3), App. D) and the damped-inverse
preconditioner (Eq. (2) step (1), App. C) against the float64 oracle.

Preconditioner inputs are spectral random SPD matrices from the input
generator, so both sides consume the same fp32 bytes of S."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,B,D", [("bf16", 37, 200), ("bf16", 16, 512), ("f32", 5, 64),
                                       ("f32", 9, 100), ("bf16", 300, 64)])
def test_cov_parity_and_symmetry(dtype, B, D):
    import torch
    import paper_2405_13954_amd as P
    from gpu_util import dev, host, normwise, say
    say(f"[cov parity] dtype={dtype} B={B} D={D}")
    g = W.normal(W.rng(21, B, D), (B, D), 1.0, dtype)
    S = torch.zeros((D, D), dtype=torch.float32, device="cuda")
    P.logra_cov_accumulate(dev(g), S)
    torch.cuda.synchronize()
    got = host(S)
    want = oracle.cov_accumulate(g)
    assert np.array_equal(got, got.T)          # exactly symmetric
    err = normwise(got, want)
    say(f"  normwise err {err:.3e}")
    assert err <= (1e-4 if dtype == "f32" else 2e-2)
    assert err <= 1e-5


def test_cov_integer_exact_blocks_and_chunks():
    import torch
    import paper_2405_13954_amd as P
    from gpu_util import dev, host, say
    say("[cov] integer exact, blocks, chunked")
    g = W.integer_array(W.rng(22), (40, 3 * 72), -3, 3, "bf16")
    S = torch.zeros((3, 72, 72), dtype=torch.float32, device="cuda")
    gd = dev(g)
    P.logra_cov_accumulate_blocks(gd[:25], S, 72)      # chunked: 25 then 15 rows
    P.logra_cov_accumulate_blocks(gd[25:], S, 72)
    torch.cuda.synchronize()
    got = host(S)
    for l in range(3):
        want = oracle.cov_accumulate(g[:, l * 72:(l + 1) * 72])
        assert np.array_equal(got[l].astype(np.float64), want)


@pytest.mark.parametrize("B1,B2,D,nb,pad,s_shift", [
    (40, 5, 192, 2, 8, 0),     # register tiles: 3 off-diagonal + 3 diagonal per block, 2 chunks then 1
    (8, 0, 128, 1, 0, 0),      # register tiles, a single short chunk
    (33, 31, 64, 3, 16, 0),    # diagonal tiles only (one tile per block)
    (20, 12, 128, 2, 0, 1),    # S not 16-byte aligned: the general kernel
])
def test_cov_integer_exact_tile_paths(B1, B2, D, nb, pad, s_shift):
    import torch
    import paper_2405_13954_amd as P
    from gpu_util import dev, host, say
    say(f"[cov] integer exact, B={B1}+{B2}, D={D}, blocks={nb}, row pad={pad}, S shift={s_shift}")
    ld = D * nb + pad
    g = W.integer_array(W.rng(24, B1, D), (B1 + B2, ld), -4, 4, "bf16")
    gd = dev(g)
    base = torch.zeros(nb * D * D + s_shift, dtype=torch.float32, device="cuda")
    S0 = W.integer_array(W.rng(25, D), (nb, D, D), -50, 50, "f32")
    S0 = S0 + S0.transpose(0, 2, 1)   # symmetric, as an accumulated S is
    base[s_shift:] = torch.from_numpy(S0.reshape(-1)).cuda()
    S = base[s_shift:].view(nb, D, D)
    for lo, hi in ((0, B1), (B1, B1 + B2)):
        if hi > lo:
            P.logra_cov_accumulate_blocks(gd[lo:hi], S, D)
    torch.cuda.synchronize()
    got = host(S)
    for l in range(nb):
        want = S0[l].astype(np.float64) + oracle.cov_accumulate(g[:, l * D:(l + 1) * D])
        assert np.array_equal(got[l].astype(np.float64), want)
        assert np.array_equal(got[l], got[l].T)


@pytest.mark.parametrize("B1,B2,D,nb,pad,dtype", [
    (40, 5, 192, 2, 8, "bf16"),    # register tiles below the diagonal + diagonal tiles, 2 chunks then 1
    (33, 0, 64, 3, 16, "bf16"),    # diagonal tiles only
    (25, 15, 72, 3, 0, "bf16"),    # ragged D: the general kernel
    (9, 4, 100, 2, 3, "f32"),      # fp32 rows: the general kernel
])
def test_cov_lower_integer_exact_upper_untouched(B1, B2, D, nb, pad, dtype):
    """Lower-triangle form (SYRK, uplo = lower): the lower triangle and diagonal
    equal the oracle's exactly; every entry above the diagonal keeps its bits."""
    import torch
    import paper_2405_13954_amd as P
    from gpu_util import dev, host, say
    say(f"[cov lower] integer exact, B={B1}+{B2}, D={D}, blocks={nb}, pad={pad}, {dtype}")
    ld = D * nb + pad
    g = W.integer_array(W.rng(26, B1, D), (B1 + B2, ld), -4, 4, dtype)
    gd = dev(g)
    S0 = W.integer_array(W.rng(27, D), (nb, D, D), -50, 50, "f32")
    S0 = S0 + S0.transpose(0, 2, 1)
    up = np.triu(np.ones((D, D), bool), 1)
    S0[:, up] = np.nan                      # never read: a NaN there would spread into the result
    S = dev(S0)
    for lo, hi in ((0, B1), (B1, B1 + B2)):
        if hi > lo:
            P.logra_cov_accumulate_blocks_lower(gd[lo:hi], S, D)
    torch.cuda.synchronize()
    got = host(S)
    assert np.array_equal(got[:, up].view(np.uint32), S0[:, up].view(np.uint32))
    for l in range(nb):
        want = S0[l].astype(np.float64) + oracle.cov_accumulate(g[:, l * D:(l + 1) * D])
        assert np.array_equal(got[l][~up].astype(np.float64), want[~up])


def test_precondition_and_self_influence_read_only_the_lower_triangle():
    """The statistic kept as its lower triangle feeds the preconditioner and the
    inverse factor to the same bits as the symmetric statistic."""
    import torch
    import paper_2405_13954_amd as P
    from gpu_util import dev, host, say
    nb, D, B, Q = 3, 128, 300, 5
    say(f"[cov lower] preconditioner and self-influence from the lower triangle, {nb} blocks of {D}")
    g = dev(W.normal(W.rng(28), (B, nb * D), 1.0, "bf16"))
    S_full = torch.zeros((nb, D, D), dtype=torch.float32, device="cuda")
    S_low = torch.triu(torch.full((nb, D, D), float("nan"), dtype=torch.float32, device="cuda"), 1)
    P.logra_cov_accumulate_blocks(g, S_full, D)
    P.logra_cov_accumulate_blocks_lower(g, S_low, D)
    torch.cuda.synchronize()
    lo = np.tril(np.ones((D, D), bool))
    assert np.array_equal(host(S_full)[:, lo].view(np.uint32), host(S_low)[:, lo].view(np.uint32))
    gt = dev(W.normal(W.rng(29), (Q, nb * D), 1.0, "f32"))
    outs = []
    for S in (S_full, S_low):
        o = torch.empty((Q, nb * D), dtype=torch.float32, device="cuda")
        P.logra_precondition_blocks(S, B, 0.1, gt, o)
        si = torch.empty(B, dtype=torch.float32, device="cuda")
        P.logra_self_influence_blocks(S, B, 0.1, g, self_out=si)
        torch.cuda.synchronize()
        outs.append((host(o), host(si)))
    assert np.all(np.isfinite(outs[0][0])) and np.all(np.isfinite(outs[0][1]))
    assert np.array_equal(outs[0][0].view(np.uint32), outs[1][0].view(np.uint32))
    assert np.array_equal(outs[0][1].view(np.uint32), outs[1][1].view(np.uint32))


def test_cov_deterministic():
    import torch
    import paper_2405_13954_amd as P
    from gpu_util import dev, host, say
    say("[cov] determinism")
    g = dev(W.normal(W.rng(23), (64, 256), 1.0, "bf16"))
    outs = []
    for _ in range(2):
        S = torch.zeros((256, 256), dtype=torch.float32, device="cuda")
        P.logra_cov_accumulate(g, S)
        torch.cuda.synchronize()
        outs.append(host(S))
    assert np.array_equal(outs[0].view(np.uint32), outs[1].view(np.uint32))


PRE_CASES = {
    # name: (D, rank, n_blocks, Q, damp, in_dtype, out_dtype)
    "tiny_f32": (64, 4, 1, 2, 1e-3, "f32", "f32"),
    "ragged_D": (200, 50, 1, 7, 0.1, "bf16", "f32"),
    "blocks_bf16": (256, 256, 5, 37, 0.1, "bf16", "bf16"),
    "blocks_many_q": (64, 30, 3, 70, 0.1, "f32", "f32"),
    "D1000": (1000, 1000, 1, 5, 0.1, "f32", "f32"),
}


@pytest.mark.parametrize("name", sorted(PRE_CASES))
def test_precondition_parity(name):
    import torch
    import paper_2405_13954_amd as P
    from gpu_util import dev, host, rowwise_normwise, say
    D, rank, nb, Q, r, idt, odt = PRE_CASES[name]
    say(f"[precondition parity] case={name}")
    N = 4096
    S = np.stack([W.spd_matrix(30 + l, D, rank, scale=float(N)) for l in range(nb)])
    g = W.normal(W.rng(31, D), (Q, nb * D), 1.0, idt)
    out = torch.zeros((Q, nb * D), dtype=torch.float32 if odt == "f32" else torch.bfloat16, device="cuda")
    P.logra_precondition_blocks(dev(S), N, r, dev(g), out)
    got = host(out)
    want = np.concatenate([oracle.precondition(S[l].astype(np.float64), N, r, g[:, l * D:(l + 1) * D])[0]
                           for l in range(nb)], axis=1)
    tol = 1e-4 if odt == "f32" else 2e-2
    for l in range(nb):
        err = rowwise_normwise(got[:, l * D:(l + 1) * D], want[:, l * D:(l + 1) * D])
        say(f"  block {l}: normwise err {err:.3e} (tol {tol})")
        assert err <= tol


def test_precondition_identity_and_single_api():
    import torch
    import paper_2405_13954_amd as P
    from gpu_util import dev, host, say
    say("[precondition] identity mode, single-block API")
    g = W.normal(W.rng(32), (3, 64), 1.0, "bf16")
    out = torch.zeros((3, 64), dtype=torch.float32, device="cuda")
    S = torch.zeros((64, 64), dtype=torch.float32, device="cuda")
    P.logra_precondition(S, 1, -1.0, dev(g), out)
    assert np.array_equal(host(out), W.bf16_bits_to_f32(g))


def test_precondition_not_pd():
    import torch
    import paper_2405_13954_amd as P
    from gpu_util import dev, say
    say("[precondition] not positive definite")
    v = np.zeros((1, 64), np.float32)
    v[0, :2] = [1.0, 2.0]
    S = np.outer(v[0], v[0]).astype(np.float32)   # rank one: second pivot is exactly zero
    out = torch.zeros((1, 64), dtype=torch.float32, device="cuda")
    with pytest.raises(P.LograError) as ei:
        P.logra_precondition(dev(S), 1, 0.0, dev(v), out)
    assert ei.value.status == P.ERR_NOT_PD
    S2 = np.eye(64, dtype=np.float32)
    S2[10, 10] = -1.0
    with pytest.raises(P.LograError) as ei:
        P.logra_precondition(dev(S2), 1, 0.0, dev(v), out)
    assert ei.value.status == P.ERR_NOT_PD
    assert "pivot 10" in P.logra_last_error()


@pytest.mark.parametrize("D,nb,Q,idt,odt", [
    (8, 3, 1, "f32", "f64"), (16, 2, 17, "f64", "f64"), (17, 1, 65, "f32", "f32"), (63, 2, 16, "bf16", "f64"),
    (65, 2, 33, "f32", "f64"), (129, 3, 5, "f32", "f64"), (255, 2, 64, "f64", "bf16"), (256, 300, 3, "bf16", "f64"),
    (256, 5, 1000, "f32", "f64"), (257, 2, 5, "f32", "f64"), (300, 1, 70, "bf16", "f32"), (512, 2, 129, "f64", "f64"),
    (777, 2, 9, "f32", "f64"), (1000, 24, 7, "f32", "f64"), (1024, 4, 64, "f32", "f64"),
    (1288, 1, 200, "bf16", "f64"),
    # 32 right-hand sides a workgroup (256 workgroups or more), the second of them with a ragged rest
    (64, 200, 45, "f32", "f64"), (40, 130, 33, "bf16", "f64"), (128, 130, 61, "f32", "f32"), (120, 130, 47, "f64", "f64"),
    (200, 130, 50, "f32", "f64"), (264, 90, 70, "f32", "f64")])
def test_precondition_panel_edges(D, nb, Q, idt, odt):
    """Widths around the 16-wide blocks, the 256-wide panels and their remainders, numbers of right-hand sides around
    the 16 and 32 of a workgroup and the 64 of a block step's tile, both solve paths, and the solve's forms for widths
    up to 64, 128 and 256 with 16 and with 32 right-hand sides a workgroup.  A float64 solve of a system of condition number kappa is
    within about D kappa 2^-53 of the oracle's; kappa <= 1 + 10 D here (damping 0.1 of the mean eigenvalue), so 1e-10
    leaves a factor of 50 at the widest; outputs in fewer bits add their rounding."""
    import torch
    import paper_2405_13954_amd as P
    from gpu_util import dev, host, rowwise_normwise, say
    say(f"[precondition panels] D={D} blocks={nb} Q={Q} in={idt} out={odt}")
    N = 50
    few = min(nb, 3)
    S = np.stack([W.spd_matrix(60 + l, D, min(D, 40), scale=float(N)) for l in range(few)])
    up = np.triu(np.ones((D, D), bool), 1)
    Sd = S.copy()
    Sd[:, up] = np.nan                       # never read
    Sd = Sd[np.arange(nb) % few]
    g = W.normal(W.rng(61, D), (Q, nb * D), 1.0, "bf16" if idt == "bf16" else "f32")
    g = g.astype(np.float64) / 3.0 if idt == "f64" else g
    out = torch.full((Q, nb * D + 3), float("nan"),
                     dtype={"f32": torch.float32, "f64": torch.float64, "bf16": torch.bfloat16}[odt], device="cuda")
    P.logra_precondition_blocks(dev(Sd), N, 0.1, dev(g), out[:, :nb * D])
    got = host(out)
    tail = got[:, nb * D:]
    assert np.isnan(W.bf16_bits_to_f32(tail) if odt == "bf16" else tail).all()
    tol = {"f64": 1e-10, "f32": 1e-6, "bf16": 5e-3}[odt]
    for l in sorted({0, 1 % nb, nb // 2, nb - 1}):
        want, _ = oracle.precondition(S[l % few].astype(np.float64), N, 0.1, np.ascontiguousarray(g[:, l * D:(l + 1) * D]))
        err = rowwise_normwise(got[:, l * D:(l + 1) * D], want)
        say(f"  block {l}: normwise err {err:.3e} (tol {tol})")
        assert err <= tol


@pytest.mark.parametrize("D,at", [(64, 0), (200, 199), (256, 100), (300, 280), (600, 511), (600, 512)])
def test_precondition_not_pd_pivot(D, at):
    """The first non-positive pivot is named, in whichever block or panel it falls."""
    import torch
    import paper_2405_13954_amd as P
    from gpu_util import dev, say
    say(f"[precondition not PD] D={D} pivot {at}")
    S = np.stack([np.eye(D, dtype=np.float32)] * 3)
    S[1, at, at] = -1.0
    S[2, at, at] = -1.0
    out = torch.zeros((2, 3 * D), dtype=torch.float32, device="cuda")
    with pytest.raises(P.LograError) as ei:
        P.logra_precondition_blocks(dev(S), 1, 0.0, dev(np.ones((2, 3 * D), np.float32)), out)
    assert ei.value.status == P.ERR_NOT_PD
    assert f"block 1: pivot {at} " in P.logra_last_error()


@pytest.mark.parametrize("D", [1, 16, 40, 256, 300, 600])
def test_precondition_infinite_damping(D):
    """lambda = inf, from an infinite damping ratio or an infinite entry on the diagonal: every solution is zero, as
    the oracle's, and no pivot is reported (inf is positive)."""
    import torch
    import paper_2405_13954_amd as P
    from gpu_util import dev, host, say
    say(f"[precondition inf] D={D}")
    S = W.spd_matrix(66, D, min(D, 40), scale=4.0)
    Sinf = S.copy()
    Sinf[D // 2, D // 2] = np.inf
    g = W.normal(W.rng(67, D), (5, D), 1.0, "f32")
    for M, damp in ((S, np.inf), (Sinf, 0.1)):
        want, lam = oracle.precondition(M.astype(np.float64), 4, damp, g)
        assert lam == np.inf and not want.any()
        for f, t in ((P.logra_precondition, torch.float32), (P.logra_precondition_f64, torch.float64)):
            out = torch.full((5, D), float("nan"), dtype=t, device="cuda")
            f(dev(M.astype(np.float32 if t == torch.float32 else np.float64)), 4, damp, dev(g), out)
            assert not host(out).any()


def test_precondition_more_right_hand_sides_than_one_grid():
    """3e8 gradients of one value: more workgroups of 32 than one launch takes."""
    import torch
    import paper_2405_13954_amd as P
    from gpu_util import say
    Q = 300_000_000
    say(f"[precondition] D=1, {Q} right-hand sides")
    S = torch.tensor([[6.0]], device="cuda")
    g = (torch.arange(Q, device="cuda", dtype=torch.int32) % 1000).to(torch.float32)[:, None]
    out = torch.full((Q, 1), float("nan"), dtype=torch.float32, device="cuda")
    P.logra_precondition(S, 2, 1.0, g, out)         # C = 3, lambda = 3
    assert (out - g / 6.0).abs().max().item() <= 1000 / 6.0 * 2.0 ** -23
