"""GPU parity of the whole Adafactor step around the decompressed gradient
(the base optimizer of the paper's experiments, Section 3.1, and its unfactored
variant, Section 3.3 "Optimizer with linear memory") against the fp64 CPU oracle:
relative step size, parameter scale carried as a sum of squares, both second
moments.  Same bars as the other update tests: 1e-5 on the fp32 matrix-core
path, 2e-2 on the bf16 path (doubled for quantities that divide two such
results), on the update W_new - W_old itself, not only on W.
"""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
from paper_2402_03293_amd import flora  # noqa: E402

pytestmark = pytest.mark.gpu

from parity_bars import TOL_BF16, TOL_F32, tol_for, update_bar  # noqa: E402,F401
DEV = "cuda:0"




def to64(t):
    return t.detach().to(torch.float32).cpu().numpy().astype(np.float64)


def rel_fro(x, ref):
    ref = np.asarray(ref, dtype=np.float64)
    x = np.asarray(x, dtype=np.float64)
    den = np.linalg.norm(ref)
    return np.linalg.norm(x - ref) / (den if den > 0 else 1.0)


def rand(shape, seed, scale=1.0):
    g = torch.Generator(device="cpu").manual_seed(seed)
    return (scale * torch.randn(*shape, generator=g)).to(DEV).contiguous()


def sync():
    torch.cuda.synchronize()


# ------------------------------------------------------------ sum of squares
def test_weight_sumsq_every_tail_and_many_matrices():
    shapes = [(1, 1), (3, 5), (7, 9), (64, 64), (257, 1023), (1000, 2050), (33, 4)]
    Ws = [rand(s, 100 + i, scale=0.5 + i) for i, s in enumerate(shapes)]
    out = torch.full((len(shapes), 4), float("nan"), device=DEV)     # one float per matrix, 16 bytes apart
    mats = flora.matrices(shapes, weights=Ws, weight_sumsqs=[out[i] for i in range(len(shapes))])
    flora.weight_sumsq(mats)
    flora.weight_sumsq(mats)        # overwrites, does not accumulate
    sync()
    got = to64(out)[:, 0]
    for i, W in enumerate(Ws):
        want = float((to64(W) ** 2).sum())
        assert got[i] == pytest.approx(want, rel=2e-6), shapes[i]
    assert torch.isnan(out[:, 1:]).all()                              # nothing else was touched


def test_schedule_helper_matches_oracle():
    for t in (1, 2, 7, 32, 1000, 10 ** 4, 40000, 10 ** 7):
        rho, beta2 = flora.adafactor_schedule(t)
        orho, obeta2 = oracle.adafactor_schedule(t)
        assert rho == pytest.approx(orho, rel=1e-6)
        assert beta2 == pytest.approx(obeta2, rel=1e-6, abs=1e-7)
    assert flora.adafactor_schedule(0) == flora.adafactor_schedule(1)


# ------------------------------------------------------- unfactored second moment
@pytest.mark.parametrize("n,m,r", [(130, 200, 16), (77, 70, 8), (300, 520, 64), (257, 264, 256), (100, 131, 128)])
@pytest.mark.parametrize("clip_d,beta2,scaled", [(0.0, 0.0, False), (1.0, 0.0, True), (0.3, 0.8, True),
                                                 (1.0, 0.9375, False)])
def test_apply_update_unfactored(n, m, r, clip_d, beta2, scaled):
    seed = 8000 + r
    S = rand((n, r), seed)
    W0 = rand((n, m), seed + 1, scale=0.05)
    V0 = (rand((n, m), seed + 2).abs() + 0.1).contiguous()
    W, V = W0.clone(), V0.clone()
    ss = torch.zeros(4, device=DEV)
    mats = flora.matrices([(n, m)], weights=[W], states=[S], seeds=[seed], second_moments=[V], weight_sumsqs=[ss])
    flora.weight_sumsq(mats)
    step, alpha, eps1, eps2 = 0.01, 0.5, 1e-30, 1e-3
    flora.apply_update(mats, r, flora.F32,
                       flora.unfactored_update(step, alpha, beta2, eps1, clip_d, scale_parameter=scaled, eps2=eps2))
    sync()
    Gt = oracle.decompress(to64(S), m, seed, alpha=alpha)
    Wr, Vr = oracle.adafactor_step(to64(W0), Gt, V=to64(V0), beta2=beta2, eps1=eps1, eps2=eps2, clip_d=clip_d,
                                   step=step, scale_parameter=scaled)
    tol = tol_for(r)
    assert rel_fro(to64(V), Vr) < tol
    dg, do = to64(W) - to64(W0), Wr - to64(W0)
    if beta2 == 0.0:
        # V = Gt^2 makes U = sign(Gt): where |Gt| is within rounding of zero the sign is not
        # determined, so those entries are only held to the size of a step
        keep = np.abs(Gt) > (0.05 if r > 32 else 1e-3) * np.sqrt((Gt ** 2).mean())
        assert keep.mean() > 0.9
        assert np.abs(dg[~keep]).max() <= 1.001 * np.abs(do).max()
        dg, do = dg[keep], do[keep]
    assert rel_fro(dg, do) < update_bar(r, Wr, to64(W0))
    # the sum of squares left behind is that of the new weights
    assert float(ss[0]) == pytest.approx(float((to64(W) ** 2).sum()), rel=5e-6)
    assert float(ss[0]) == pytest.approx(float((Wr ** 2).sum()), rel=tol)


def test_unfactored_first_step_is_sign_descent_on_the_gpu():
    # beta2 = 0, tiny eps1: U = sign(Gt), RMS(U) = 1, so W moves by exactly step * RMS(W) per entry
    n, m, r, seed = 96, 160, 32, 31
    S = rand((n, r), seed)
    W0 = torch.full((n, m), -2.0, device=DEV)
    W, V = W0.clone(), torch.zeros((n, m), device=DEV)
    ss = torch.zeros(4, device=DEV)
    mats = flora.matrices([(n, m)], weights=[W], states=[S], seeds=[seed], second_moments=[V], weight_sumsqs=[ss])
    flora.weight_sumsq(mats)
    flora.apply_update(mats, r, flora.F32, flora.unfactored_update(0.01, 1.0, 0.0, 1e-30, 1.0, scale_parameter=True))
    sync()
    d = to64(W) - to64(W0)
    np.testing.assert_allclose(np.abs(d), 0.02, rtol=1e-5)
    Gt = oracle.decompress(to64(S), m, seed, alpha=1.0)
    big = np.abs(Gt) > 1e-3 * np.abs(Gt).max()
    assert np.array_equal(np.sign(d)[big], -np.sign(Gt)[big])


# ------------------------------------------------------- the reduction passes by products of bf16 parts (r = 16)
# State entries beyond the largest bf16 value have no parts, and tiles with one are multiplied in fp32: statistics and
# weights come out as of any other state (alpha brings the product back), and an infinity's row and the columns' sums are infinite.
# No clipping: its sum takes alpha^2, which is below fp32's range here.
@pytest.mark.parametrize("n,m", [(1, 5), (70, 129), (33, 300)])
@pytest.mark.parametrize("r", [16, 32])
def test_factored_passes_of_states_beyond_bf16(n, m, r):
    seed, alpha, big = 77, 2e-38, sorted({0, n // 2, n - 1})
    A = oracle.materialise_A(seed, m, r)
    cols = [int(k) for k in np.argsort(np.abs(A).max(axis=0))[:len(big)]]
    S = rand((n, r), 5, scale=2e37)
    for i, k in zip(big, cols):
        assert np.abs(A[:, k]).max() < 1.0                   # (or the product itself overflows)
        S[i] = 0
        S[i, k] = 3.4e38 * (-1) ** i
    W0, R0, K0 = rand((n, m), 6), rand((n,), 7).abs() + 0.5, rand((m,), 8).abs() + 0.5
    W, R, K = W0.clone(), R0.clone(), K0.clone()
    mats = flora.matrices([(n, m)], weights=[W], states=[S], row_stats=[R], col_stats=[K], seeds=[seed])
    flora.apply_update(mats, r, flora.F32, flora.factored_update(1e-2, alpha, 0.5, 1e-30, 0.0))
    sync()
    Wr, Rr, Kr = oracle.factored_update(to64(W0), oracle.decompress(to64(S), m, seed, alpha=alpha), to64(R0), to64(K0), 0.5, 1e-30, 0.0, 1e-2)
    assert rel_fro(to64(R), Rr) < TOL_F32 and rel_fro(to64(K), Kr) < TOL_F32
    assert rel_fro(to64(W) - to64(W0), Wr - to64(W0)) < update_bar(r, Wr, to64(W0))
    # an infinity
    S[big[-1], cols[-1]] = float("inf")
    R, K = R0.clone(), K0.clone()
    mats = flora.matrices([(n, m)], weights=[W.clone()], states=[S], row_stats=[R], col_stats=[K], seeds=[seed])
    flora.apply_update(mats, r, flora.F32, flora.factored_update(1e-2, alpha, 0.5, 1e-30, 0.0))
    sync()
    assert np.isposinf(to64(R)[big[-1]]) and np.isposinf(to64(K)).all()
    rest = [i for i in range(n) if i != big[-1]]
    assert rel_fro(to64(R)[rest], Rr[rest]) < TOL_F32


# ------------------------------------------------ several steps with the carried scale
@pytest.mark.parametrize("r,rule", [(16, "factored"), (64, "factored"), (256, "unfactored"), (32, "unfactored")])
def test_adafactor_steps_with_schedules_and_carried_parameter_scale(r, rule):
    shapes = [(96, 200), (130, 64), (40, 520)]
    count = len(shapes)
    W = [rand(s, 300 + i, scale=0.02 * (i + 1)) for i, s in enumerate(shapes)]
    St = [torch.zeros((n, r), device=DEV) for (n, m) in shapes]
    R = [torch.zeros(n, device=DEV) for (n, m) in shapes]
    K = [torch.zeros(m, device=DEV) for (n, m) in shapes]
    # the unfactored second moment starts from a typical magnitude (Gt^2 is about m / r here): from
    # zero the first steps would be sign(Gt), whose value near Gt = 0 no tolerance can pin
    V = [torch.full(s, float(s[1]) / r, device=DEV) for s in shapes]
    ss = torch.zeros((count, 4), device=DEV)
    Wo = [to64(w) for w in W]
    Ro = [np.zeros(n) for (n, m) in shapes]
    Ko = [np.zeros(m) for (n, m) in shapes]
    Vo = [to64(v) for v in V]
    gdt = torch.float32 if r <= 32 else torch.bfloat16
    eps1, eps2 = 1e-30, 1e-3
    kw = dict(weights=W, states=St, weight_sumsqs=[ss[i] for i in range(count)])
    if rule == "factored":
        kw.update(row_stats=R, col_stats=K)
    else:
        kw.update(second_moments=V)
    flora.weight_sumsq(flora.matrices(shapes, **kw))           # once; the updates carry it afterwards
    for t in range(1, 5):
        seeds = [int(flora.derive_seed(9, l, t)) for l in range(count)]
        G = [rand(s, 1000 * t + i).to(gdt).contiguous() for i, s in enumerate(shapes)]
        mats = flora.matrices(shapes, grads=G, seeds=seeds, **kw)
        flora.compress(mats, r, flora.F32 if r <= 32 else flora.BF16, 1.0, 1.0)
        prev = [to64(w) for w in W]
        rho, beta2 = flora.adafactor_schedule(t)
        mk = flora.factored_update if rule == "factored" else flora.unfactored_update
        flora.apply_update(mats, r, flora.F32, mk(rho, 1.0, beta2, eps1, 1.0, zero_state_after=True,
                                                  scale_parameter=True, eps2=eps2))
        sync()
        orho, obeta2 = oracle.adafactor_schedule(t)
        for l, (n, m) in enumerate(shapes):
            C = oracle.compress(to64(G[l]), r, seeds[l])
            Gt = oracle.decompress(C, m, seeds[l], alpha=1.0)
            before = Wo[l]
            if rule == "factored":
                Wo[l], Ro[l], Ko[l] = oracle.adafactor_step(before, Gt, R=Ro[l], K=Ko[l], beta2=obeta2, eps1=eps1,
                                                            eps2=eps2, step=orho)
            else:
                Wo[l], Vo[l] = oracle.adafactor_step(before, Gt, V=Vo[l], beta2=obeta2, eps1=eps1, eps2=eps2,
                                                     step=orho)
            tol = tol_for(r)
            # this step's movement on either side (the two trajectories stay within the bar of
            # each other, so second moments and parameter scales agree to the same order)
            dg, do = to64(W[l]) - prev[l], Wo[l] - before
            if rule == "unfactored" and obeta2 == 0.0:
                # the schedule's first step has beta2 = 0: V = Gt^2 and U = sign(Gt), whose value
                # where |Gt| is within rounding of zero no tolerance can pin (see the single-step
                # test above): those entries are held to the size of a step, the rest to the bar
                keep = np.abs(Gt) > (0.05 if r > 32 else 1e-3) * np.sqrt((Gt ** 2).mean())
                assert keep.mean() > 0.9
                assert np.abs(dg[~keep]).max() <= 1.001 * np.abs(do).max()
                dg, do = dg[keep], do[keep]
            assert rel_fro(dg, do) < update_bar(r, Wo[l], before), (t, l)
            assert rel_fro(to64(W[l]), Wo[l]) < (1e-6 if r <= 32 else tol), (t, l)
            assert float(ss[l, 0]) == pytest.approx(float((Wo[l] ** 2).sum()), rel=tol), (t, l)
        assert float(max(s.abs().max() for s in St)) == 0.0


# both bf16 decompress kernels, one and several row blocks per matrix
@pytest.mark.parametrize("vec", [1, 2])
@pytest.mark.parametrize("rows", [0, 64])
@pytest.mark.parametrize("n,m,r", [(300, 520, 64), (257, 264, 256), (200, 1028, 128)])
def test_bf16_kernels_unfactored_and_scaled_factored(n, m, r, rows, vec):
    seed = 9000 + n + r
    S = rand((n, r), seed)
    W0 = rand((n, m), seed + 1, scale=0.1)
    V0 = (rand((n, m), seed + 2).abs() + 0.1).contiguous()
    R0 = (rand((n,), seed + 3).abs() + 0.1).contiguous()
    K0 = (rand((m,), seed + 4).abs() + 0.1).contiguous()
    step, alpha, eps1, eps2, beta2, clip_d = 0.01, 0.5, 1e-30, 1e-3, 0.8, 0.3
    Wu, Wf, V, R, K = W0.clone(), W0.clone(), V0.clone(), R0.clone(), K0.clone()
    ssu, ssf = torch.zeros(4, device=DEV), torch.zeros(4, device=DEV)
    flora.set_tuning("decompress_vec", vec)
    flora.set_tuning("decompress_rows", rows)
    try:
        mu = flora.matrices([(n, m)], weights=[Wu], states=[S], seeds=[seed], second_moments=[V], weight_sumsqs=[ssu])
        mf = flora.matrices([(n, m)], weights=[Wf], states=[S], seeds=[seed], row_stats=[R], col_stats=[K],
                            weight_sumsqs=[ssf])
        flora.weight_sumsq(mu)
        flora.weight_sumsq(mf)
        flora.apply_update(mu, r, flora.F32, flora.unfactored_update(step, alpha, beta2, eps1, clip_d,
                                                                     scale_parameter=True, eps2=eps2))
        flora.apply_update(mf, r, flora.F32, flora.factored_update(step, alpha, beta2, eps1, clip_d,
                                                                   scale_parameter=True, eps2=eps2))
        sync()
    finally:
        flora.set_tuning("decompress_vec", 0)
        flora.set_tuning("decompress_rows", 0)
    Gt = oracle.decompress(to64(S), m, seed, alpha=alpha)
    Wr, Vr = oracle.adafactor_step(to64(W0), Gt, V=to64(V0), beta2=beta2, eps1=eps1, eps2=eps2, clip_d=clip_d,
                                   step=step)
    assert rel_fro(to64(V), Vr) < TOL_BF16
    # row by row: a misplaced tile would hide in the norm of the whole
    dV = to64(V) - Vr
    assert (np.linalg.norm(dV, axis=1) / np.linalg.norm(Vr, axis=1)).max() < TOL_BF16
    assert rel_fro(to64(Wu) - to64(W0), Wr - to64(W0)) < TOL_BF16
    assert float(ssu[0]) == pytest.approx(float((to64(Wu) ** 2).sum()), rel=5e-6)
    Wr, Rr, Kr = oracle.adafactor_step(to64(W0), Gt, R=to64(R0), K=to64(K0), beta2=beta2, eps1=eps1, eps2=eps2,
                                       clip_d=clip_d, step=step)
    assert rel_fro(to64(R), Rr) < TOL_BF16
    assert rel_fro(to64(K), Kr) < TOL_BF16
    assert rel_fro(to64(Wf) - to64(W0), Wr - to64(W0)) < TOL_BF16
    assert float(ssf[0]) == pytest.approx(float((to64(Wf) ** 2).sum()), rel=5e-6)


def test_parameter_scale_floor_and_no_sumsq_pointer():
    # W = 0: the scale is eps2; without scale_parameter no weight_sumsq is needed
    n, m, r, seed = 64, 96, 16, 5
    S = rand((n, r), seed)
    W = torch.zeros((n, m), device=DEV)
    V = torch.zeros((n, m), device=DEV)
    ss = torch.zeros(4, device=DEV)
    mats = flora.matrices([(n, m)], weights=[W], states=[S], seeds=[seed], second_moments=[V], weight_sumsqs=[ss])
    flora.apply_update(mats, r, flora.F32, flora.unfactored_update(0.01, 1.0, 0.0, 1e-30, 1.0,
                                                                   scale_parameter=True, eps2=1e-3))
    sync()
    np.testing.assert_allclose(np.abs(to64(W)), 1e-5, rtol=1e-5)
    W2 = torch.zeros((n, m), device=DEV)
    V2 = torch.zeros((n, m), device=DEV)
    mats = flora.matrices([(n, m)], weights=[W2], states=[S], seeds=[seed], second_moments=[V2])
    flora.apply_update(mats, r, flora.F32, flora.unfactored_update(0.25, 1.0, 0.0, 1e-30, 1.0))
    sync()
    np.testing.assert_allclose(np.abs(to64(W2)), 0.25, rtol=1e-5)


def test_adafactor_argument_errors_launch_nothing():
    n, m, r = 32, 32, 16
    S = rand((n, r), 1)
    W = rand((n, m), 2)
    W0 = W.clone()
    V = torch.zeros((n, m), device=DEV)
    lib = flora.lib()
    import ctypes

    def status(mats, upd):
        return lib.flora_apply_update(mats, len(mats), r, flora.F32, ctypes.byref(upd), None)

    no_v = flora.matrices([(n, m)], weights=[W], states=[S], seeds=[1])
    assert status(no_v, flora.unfactored_update(0.1, 1.0, 0.0, 1e-30, 1.0)) == flora.ERR_INVALID
    with_v = flora.matrices([(n, m)], weights=[W], states=[S], seeds=[1], second_moments=[V])
    assert status(with_v, flora.unfactored_update(0.1, 1.0, 0.0, 1e-30, 1.0, scale_parameter=True)) == flora.ERR_INVALID
    assert status(with_v, flora.unfactored_update(0.1, 1.0, 1.5, 1e-30, 1.0)) == flora.ERR_INVALID
    alias = flora.matrices([(n, m)], weights=[W], states=[S], seeds=[1], second_moments=[W])
    assert status(alias, flora.unfactored_update(0.1, 1.0, 0.0, 1e-30, 1.0)) == flora.ERR_INVALID
    assert lib.flora_weight_sumsq(with_v, 1, flora.F32, None) == flora.ERR_INVALID      # no weight_sumsq pointer
    sync()
    assert torch.equal(W, W0)
    assert float(V.abs().max()) == 0.0


# ------------------------------------------------------------------ bf16 weights
def bf16_round(x):
    """fp64 -> nearest bf16 (ties to even), through fp32 as the kernels do."""
    u = np.asarray(x, dtype=np.float32).view(np.uint32).astype(np.uint64)
    u = (u + 0x7FFF + ((u >> 16) & 1)) >> 16 << 16
    return u.astype(np.uint32).view(np.float32).astype(np.float64)


@pytest.mark.parametrize("n,m,r", [(130, 200, 16), (77, 70, 8), (300, 520, 64), (257, 264, 256), (100, 131, 128)])
@pytest.mark.parametrize("rule", ["sgd", "factored", "unfactored"])
def test_updates_on_bf16_weights(n, m, r, rule):
    # the update is computed in fp32 from the bf16 weights and rounded when stored: against the
    # oracle's result rounded the same way the stored weights may differ by one bf16 step where
    # the exact value falls next to a rounding boundary, and nowhere by more
    seed = 9500 + r
    S = rand((n, r), seed)
    W0 = rand((n, m), seed + 1, scale=0.5).to(torch.bfloat16).contiguous()
    W = W0.clone()
    ss = torch.zeros(4, device=DEV)
    kw = dict(weights=[W], states=[S], seeds=[seed], weight_sumsqs=[ss])
    lr, alpha = 0.05, 0.5
    Gt = oracle.decompress(to64(S), m, seed, alpha=alpha)
    W064 = to64(W0)
    if rule == "sgd":
        mats = flora.matrices([(n, m)], **kw)
        flora.apply_update(mats, r, flora.BF16, flora.sgd_update(lr, alpha))
        Wr = oracle.sgd(W064, Gt, lr)
    elif rule == "factored":
        R, K = torch.zeros(n, device=DEV), torch.zeros(m, device=DEV)
        mats = flora.matrices([(n, m)], row_stats=[R], col_stats=[K], **kw)
        flora.weight_sumsq(mats, flora.BF16)
        flora.apply_update(mats, r, flora.BF16, flora.factored_update(lr, alpha, 0.0, 1e-30, 1.0, scale_parameter=True))
        Wr, _, _ = oracle.adafactor_step(W064, Gt, R=np.zeros(n), K=np.zeros(m), beta2=0.0, step=lr)
    else:
        V0 = (rand((n, m), seed + 2).abs() + 0.1).contiguous()
        V = V0.clone()
        mats = flora.matrices([(n, m)], second_moments=[V], **kw)
        flora.weight_sumsq(mats, flora.BF16)
        flora.apply_update(mats, r, flora.BF16, flora.unfactored_update(lr, alpha, 0.8, 1e-30, 1.0, scale_parameter=True))
        Wr, Vr = oracle.adafactor_step(W064, Gt, V=to64(V0), beta2=0.8, step=lr)
        assert rel_fro(to64(V), Vr) < tol_for(r)
    sync()
    assert W.dtype == torch.bfloat16
    got, want = to64(W), bf16_round(Wr)
    dg, do = got - W064, Wr - W064
    # one bf16 step at that magnitude, plus what the path's own error can move a value
    step = np.maximum(np.abs(want), np.abs(got)) * 2.0 ** -7 + tol_for(r) * np.abs(do).max()
    assert (np.abs(got - want) <= step).all()
    # the movement itself, where it is well above the rounding of the weights
    big = np.abs(do) > 8 * np.abs(W064) * 2.0 ** -8
    if big.sum() > 100:
        assert rel_fro(dg[big], do[big]) < 0.1
    mismatches = (got != want).mean()
    assert mismatches < (0.002 if r <= 32 else 0.08), mismatches
    if rule != "sgd":
        assert float(ss[0]) == pytest.approx(float((got ** 2).sum()), rel=5e-6)   # of the stored values


def test_weight_sumsq_bf16_and_vector_kernel_tails():
    shapes = [(3, 5), (64, 64), (257, 1023), (33, 4)]
    Ws = [rand(s, 200 + i).to(torch.bfloat16).contiguous() for i, s in enumerate(shapes)]
    out = torch.zeros((len(shapes), 4), device=DEV)
    mats = flora.matrices(shapes, weights=Ws, weight_sumsqs=[out[i] for i in range(len(shapes))])
    flora.weight_sumsq(mats, flora.BF16)
    sync()
    for i, W in enumerate(Ws):
        assert float(out[i, 0]) == pytest.approx(float((to64(W) ** 2).sum()), rel=2e-6)


# the cache policy of the weights (plain / streamed reads / streamed writes / both) is a hint to the
# memory system and nothing else: every policy gives the same bits, for every rule, in the 4-byte
# and the 16-byte-per-lane kernels
@pytest.mark.parametrize("rule", ["sgd", "factored", "unfactored"])
@pytest.mark.parametrize("n,m,r,wdt", [(130, 200, 16, "f32"), (97, 1001, 64, "f32"), (257, 264, 256, "f32"),
                                       (257, 264, 128, "bf16"), (70, 130, 32, "bf16")])
def test_update_cache_policies_give_the_same_bits(n, m, r, wdt, rule):
    dt = torch.float32 if wdt == "f32" else torch.bfloat16
    fd = flora.F32 if wdt == "f32" else flora.BF16
    seed = 5100 + n + m + r
    g = torch.Generator(device="cpu").manual_seed(seed)
    W0 = torch.randn(n, m, generator=g).to(dt).to(DEV)
    S = torch.randn(n, r, generator=g).to(DEV)
    out = []
    for policy in (1, 2, 3, 4):
        W = W0.clone()
        kw = dict(weights=[W], states=[S.clone()], seeds=[seed])
        if rule == "factored":
            kw.update(row_stats=[torch.zeros(n, device=DEV)], col_stats=[torch.zeros(m, device=DEV)])
            upd = flora.factored_update(1e-2, 1.0, 0.0, 1e-30, 1.0)
        elif rule == "unfactored":
            kw.update(second_moments=[torch.full((n, m), 0.5, device=DEV)])
            upd = flora.unfactored_update(1e-2, 1.0, 0.5, 1e-30, 1.0)
        else:
            upd = flora.sgd_update(1e-2, 1.0)
        flora.set_tuning("update_wpolicy", policy)
        try:
            flora.apply_update(flora.matrices([(n, m)], **kw), r, fd, upd)
            torch.cuda.synchronize()
        finally:
            flora.set_tuning("update_wpolicy", 0)
        out.append(W.clone())
        assert not torch.equal(W, W0)
    for W in out[1:]:
        assert torch.equal(W, out[0])


# the unfactored rule's second pass takes the table from its end in sets above 192 MiB, 256 with bf16 weights (a set's share of
# such a step here), unless a tenth or more of the elements are in rows off line boundaries: the same bits, whichever order
@pytest.mark.parametrize("r,wdt", [(16, "f32"), (32, "bf16"), (64, "f32"), (256, "bf16")])
@pytest.mark.parametrize("shapes,reverse", [([(130, 256), (33, 512), (257, 64), (5, 35)], 1), ([(97, 1001), (64, 35)], 0)])
def test_unfactored_second_pass_from_the_end(shapes, reverse, r, wdt):
    dt, fd = (torch.float32, flora.F32) if wdt == "f32" else (torch.bfloat16, flora.BF16)
    W0 = [rand(s, 300 + i).to(dt).contiguous() for i, s in enumerate(shapes)]
    S = [rand((n, r), 310 + i) for i, (n, _) in enumerate(shapes)]
    out = []
    for mib, policy in ((0.0, (0, 0, 0, 0)), (257.0, (0, 3, 1, 0) if reverse else (0, 0, 0, 0))):
        W, V = [w.clone() for w in W0], [torch.full(s, 0.5, device=DEV) for s in shapes]
        sq = [torch.ones(1, device=DEV) for _ in shapes]
        mats = flora.matrices(shapes, weights=W, states=S, second_moments=V, weight_sumsqs=sq, seeds=[7, 8, 9, 10][:len(shapes)])
        u = flora.unfactored_update(1e-2, 1.0, 0.5, 1e-30, 1.0, step_weight_mib=mib)
        assert flora.debug_access_policy(mats, r, fd, u) == policy
        flora.apply_update(mats, r, fd, u)
        sync()
        out.append(W + V + sq)
    assert all(torch.equal(x, y) for x, y in zip(*out))
    assert not torch.equal(out[0][0], W0[0])


# ------------------------------------------- the factored rule through Gram matrices
# Row sums, column sums and the clipping sum of the rule as quadratic forms in A^T A, S^T S and
# A^T diag(1/K) A (ranks >= 64), against the oracle, and against the passes over the decompressed
# gradient that they replace: ragged shapes, many pieces of the Gram sums (a few tiles of 64 each, as in any short
# launch), several blocks of rows and columns of the quadratic forms (256, and 256 or 512), grouped
# matrices, with and without clipping.  The next two tests take the long loops.
@pytest.mark.parametrize("r", [64, 128, 256])
@pytest.mark.parametrize("clip_d,beta2", [(1.0, 0.0), (0.0, 0.6), (0.3, 0.8)])
def test_factored_rule_through_gram_matrices(r, clip_d, beta2):
    shapes = [(300, 520), (130, 6500), (3300, 264), (64, 64), (1100, 1032)]
    count = len(shapes)
    g = torch.Generator(device="cpu").manual_seed(900 + r)
    S = [torch.randn(n, r, generator=g).to(DEV) for n, _ in shapes]
    W0 = [torch.randn(*s, generator=g).to(DEV) for s in shapes]
    R0 = [(torch.rand(n, generator=g) + 0.5).to(DEV) for n, _ in shapes]
    K0 = [(torch.rand(m, generator=g) + 0.5).to(DEV) for _, m in shapes]
    seeds = [int(flora.derive_seed(77, l, r)) for l in range(count)]
    lr, alpha, eps1 = 0.01, 0.5, 1e-30
    res = {}
    for mode in (1, 2):
        W, R, K = [x.clone() for x in W0], [x.clone() for x in R0], [x.clone() for x in K0]
        flora.set_tuning("factored_gram", mode)
        try:
            mats = flora.matrices(shapes, weights=W, states=S, row_stats=R, col_stats=K, seeds=seeds)
            flora.apply_update(mats, r, flora.F32, flora.factored_update(lr, alpha, beta2, eps1, clip_d))
            sync()
        finally:
            flora.set_tuning("factored_gram", 0)
        res[mode] = (W, R, K)
    for l, (n, m) in enumerate(shapes):
        Gt = oracle.decompress(to64(S[l]), m, seeds[l], alpha=alpha)
        Wr, Rr, Kr = oracle.factored_update(to64(W0[l]), Gt, to64(R0[l]), to64(K0[l]), beta2, eps1, clip_d, lr)
        for mode in (1, 2):
            W, R, K = res[mode]
            assert rel_fro(to64(R[l]), Rr) < TOL_BF16, (mode, shapes[l])
            assert rel_fro(to64(K[l]), Kr) < TOL_BF16, (mode, shapes[l])
            assert rel_fro(to64(W[l]) - to64(W0[l]), Wr - to64(W0[l])) < TOL_BF16, (mode, shapes[l])
        # the two routes agree far more closely with each other than either must with the oracle
        assert rel_fro(to64(res[2][1][l]), to64(res[1][1][l])) < 2e-3
        assert rel_fro(to64(res[2][2][l]), to64(res[1][2][l])) < 2e-3
        e = rel_fro(to64(res[2][1][l]), Rr)
        print("gram route r=%d %s: R err %.2e K err %.2e" % (r, shapes[l], e, rel_fro(to64(res[2][2][l]), Kr)))


# The route (Gram matrices or passes) may not depend on how many matrices share the call: the statistics of one
# matrix stepped alone, with 3 and with 15 others of its shape.  Between calls only the pieces of the fp32 sums
# differ (1e-6), which turns a few bf16 roundings of Gram entries (2^-9 each, on a share of about 1e-3 of the
# r^2 terms of a quadratic form: 2^-9 sqrt(1e-3) / r < 1e-6); the two routes are 2e-4 apart at least.
@pytest.mark.parametrize("n,m,r", [(768, 3072, 128), (512, 2048, 64), (1600, 2048, 256)])
def test_factored_statistics_do_not_depend_on_the_number_of_matrices(n, m, r):
    g = torch.Generator(device="cpu").manual_seed(r)
    S = torch.randn(n, r, generator=g).to(DEV)
    W0 = torch.randn(n, m, generator=g).to(DEV)
    got = []
    for count in (1, 4, 16):
        Ws, Ss = [W0.clone() for _ in range(count)], [S.clone() for _ in range(count)]
        R = [torch.full((n,), 0.5, device=DEV) for _ in range(count)]
        K = [torch.full((m,), 0.5, device=DEV) for _ in range(count)]
        mats = flora.matrices([(n, m)] * count, weights=Ws, states=Ss, row_stats=R, col_stats=K, seeds=[9] * count)
        flora.apply_update(mats, r, flora.F32, flora.factored_update(1e-2, 1.0, 0.2, 1e-30, 1.0))
        sync()
        got.append((to64(R[0]), to64(K[0]), to64(Ws[0]) - to64(W0)))
    for one in got[1:]:
        for a, b in zip(one, got[0]):
            assert rel_fro(a, b) < 2e-5


# Gram sums in pieces of 3072 (the loops over tiles at their longest, and a last piece that is short)
@pytest.mark.parametrize("r", [64, 128, 256])
@pytest.mark.parametrize("clip_d,beta2", [(1.0, 0.0), (0.0, 0.6)])
def test_factored_rule_through_gram_matrices_in_large_pieces(r, clip_d, beta2):
    flora.set_tuning("gram_chunk", 3072)
    try:
        test_factored_rule_through_gram_matrices(r, clip_d, beta2)
    finally:
        flora.set_tuning("gram_chunk", 0)


# ... and in pieces whose number puts P and P' on blocks of 32 ranks (up to 25 pieces at r = 128, 7 at r = 256), of 64 (up to
# 48 at r = 256), and on whole matrices (29 pieces of 320 at r = 128, 69 of 128 at r = 256): pieces that end within a tile,
# within a round of the groups' tiles, and of one tile
@pytest.mark.parametrize("r,chunk", [(128, 512), (128, 1216), (128, 320), (256, 576), (256, 768), (256, 256), (256, 192), (256, 128)])
@pytest.mark.parametrize("clip_d,beta2", [(1.0, 0.0), (0.0, 0.6)])
def test_factored_rule_through_blocks_of_gram_matrices(r, chunk, clip_d, beta2):
    flora.set_tuning("gram_chunk", chunk)
    try:
        test_factored_rule_through_gram_matrices(r, clip_d, beta2)
    finally:
        flora.set_tuning("gram_chunk", 0)


# Column statistics in blocks of 1024 columns: a set with 384 such blocks (several rounds of rows of A per workgroup,
# the last of a matrix short)
@pytest.mark.parametrize("r", [64, 128, 256])
def test_factored_rule_through_gram_matrices_with_large_column_blocks(r):
    n, m, count = 40, 4000, 100
    g = torch.Generator(device="cpu").manual_seed(950 + r)
    S, W0 = torch.randn(count, n, r, generator=g).to(DEV), torch.randn(count, n, m, generator=g).to(DEV)
    W, R, K = W0.clone(), torch.full((count, n), 0.7, device=DEV), torch.full((count, m), 0.6, device=DEV)
    seeds = [int(flora.derive_seed(78, l, r)) for l in range(count)]
    flora.set_tuning("factored_gram", 2)
    try:
        mats = flora.matrices([(n, m)] * count, weights=list(W), states=list(S), row_stats=list(R), col_stats=list(K), seeds=seeds)
        flora.apply_update(mats, r, flora.F32, flora.factored_update(0.01, 0.5, 0.4, 1e-30, 1.0))
        sync()
    finally:
        flora.set_tuning("factored_gram", 0)
    for l in (0, 57, count - 1):
        Gt = oracle.decompress(to64(S[l]), m, seeds[l], alpha=0.5)
        Wr, Rr, Kr = oracle.factored_update(to64(W0[l]), Gt, np.full(n, 0.7), np.full(m, 0.6), 0.4, 1e-30, 1.0, 0.01)
        assert rel_fro(to64(R[l]), Rr) < TOL_BF16 and rel_fro(to64(K[l]), Kr) < TOL_BF16, l
        assert rel_fro(to64(W[l]) - to64(W0[l]), Wr - to64(W0[l])) < TOL_BF16, l
