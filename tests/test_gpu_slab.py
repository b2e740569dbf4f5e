"""The slab kernels (bf16: source side -> coefficient-major workspace -> destination side) at the sizes where
they can go wrong: token counts around a slab of 64 and a group of 16, blocks applied directly, in one
radix-4 stage and in several, on either side, groups with a remainder, several slabs per dC partial row, and
calls split over the workspace.  Backwards run here throughout (frames in several stages: past the generic
kernels' token counts), forwards where the support is dense enough or the call long enough for the
dispatch's line; the others cover the generic forward at the same sizes.  Element-wise bounds against the
oracle as in the other parity tests."""
import numpy as np
import pytest

from paper_2608_26430_amd import inputs
from tests.parity_util import BwdBounds, FwdBounds, guarded, guards_intact, oracle_frame, plan_c, to_np, torch_act, user_dc, within

torch = pytest.importorskip("torch")
import paper_2608_26430_amd as ff  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    return torch.device("cuda:0")


def _ok(name, got, ref, bound):
    ok, worst = within(got, ref, bound)
    assert ok, f"{name}: element-wise bound exceeded (max err/bound {worst:.3g})"


# (n, rho_in, m, rho_out, nnz, T): 32-wide blocks; 8-wide ones, 24 x 8 rows a remainder of 64-row groups;
# 344-wide factored ones on both sides, and with direct ones on either; several stages: 4^2 x 17 and
# 4^2 x 20 (two stages), 4^3 x 17 (three), beyond the generic kernels' token counts; 16500 tokens: two slabs
# per dC partial row; and last, wide enough that the shortest forwards take the slab kernels too
CASES = [(2048, 128, 2048, 128, 30000, t) for t in (1, 15, 63, 64, 65)] + [
    (520, 130, 1032, 258, 30000, 81),
    (2752, 16, 2752, 16, 30000, 70),
    (2752, 16, 2048, 32, 40000, 129),
    (2048, 32, 2752, 16, 40000, 17),
    (544, 2, 544, 2, 700, 5009),
    (640, 2, 640, 2, 900, 4449),
    (2176, 2, 2176, 2, 3000, 2561),
    (256, 16, 256, 16, 600, 16500),
] + [(2048, 128, 4096, 256, 60000, t) for t in (1, 15, 63, 64, 65)]
# the other shapes of the DFT of size k2 in two stages (k2 = 32, 36, 44, 52, 60) and in three (32), each just past
# the generic kernels' token counts; two blocks in two stages; and a block in two stages with directly applied
# and factored ones on the other side; and the longest calls that still run in the generic kernels
STAGES = [(1024, 2, 1024, 2, 1500, 3401), (1024, 2, 1024, 2, 1500, 2271), (1152, 2, 1152, 2, 1500, 3217), (1408, 2, 1408, 2, 1500, 2961),
          (1664, 2, 1664, 2, 1500, 2785), (1920, 2, 1920, 2, 1500, 2657), (4096, 2, 4096, 2, 3000, 2209),
          (2176, 4, 2176, 4, 2000, 2561), (1152, 2, 768, 64, 1500, 3489), (688, 4, 1152, 2, 1500, 3569)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "n%d_m%d_nnz%d_T%d" % (c[0], c[2], c[4], c[5]))
def test_slab_parity(dev, case):
    n, rn, m, rm, nnz, T = case
    g = inputs.rng(n + 3 * m + T)
    _parity(dev, n, rn, m, rm, *inputs.support(g, m, n, nnz), T, g)


@pytest.mark.parametrize("case", STAGES, ids=lambda c: "n%d_m%d_nnz%d_T%d" % (c[0], c[2], c[4], c[5]))
def test_slab_parity_several_stages(dev, case):
    """As above; the tokens that are not compared are zero, so that the oracle's dC takes those alone."""
    n, rn, m, rm, nnz, T = case
    g = inputs.rng(n + 3 * m + T)
    _parity(dev, n, rn, m, rm, *inputs.support(g, m, n, nnz), T, g, few=True)


# rows and columns of very different lengths, whose entries share a step among several lanes: blocks applied
# directly, in one radix-4 stage and in two, on either side
@pytest.mark.parametrize("case", [(520, 130, 1032, 258, 81), (2752, 16, 2048, 32, 65), (2048, 32, 2752, 16, 70),
                                  (544, 2, 544, 2, 5009)], ids=lambda c: "n%d_m%d_T%d" % (c[0], c[2], c[4]))
def test_slab_uneven_supports(dev, case):
    n, rn, m, rm, T = case
    g = inputs.rng(n + m)
    C = np.zeros((m, n), dtype=bool)
    C[:, :rn:8] = True          # a dense column in every fourth block (canonical order runs through the blocks)
    C[1:rm:16] = True           # a dense row in every eighth
    C[:, 1] = g.random(m) < 0.2
    C[g.integers(0, m, 200), g.integers(0, n, 200)] = True
    rows, cols = np.nonzero(C)
    p = g.permutation(rows.size)
    _parity(dev, n, rn, m, rm, rows[p].astype(np.int32), cols[p].astype(np.int32), T, g)


def _parity(dev, n, rn, m, rm, rows, cols, T, g, few=False):
    k_in, k_out, s, nnz = n // rn, m // rm, 0.173, rows.size
    vals = inputs.gaussian(g, (nnz,), std=0.02)
    X, G = inputs.gaussian(g, (T, n), dtype="bf16"), inputs.gaussian(g, (T, m), dtype="bf16")
    # rows are independent of one another: the edges of the calls' slabs and groups, and some between
    e = 5 if few else 20
    t = np.unique(np.concatenate([np.arange(min(T, e)), np.arange(max(0, T - e), T),
                                  np.clip([47, 48, 63, 64, 127, 128], 0, T - 1), inputs.rng(T).integers(0, T, e)]))
    if few:
        zero = np.setdiff1d(np.arange(T), t)
        X[zero] = G[zero] = 0
    plan = ff.plan_create(ff.framegen(n, k_in, rn), ff.framegen(m, k_out, rm), rows, cols, max_tokens=T)
    assert not plan.fast128
    _, Xd = guarded(T, n, n + 8, "bf16", dev, X)
    _, Gd = guarded(T, m, m + 16, "bf16", dev, G)
    ybuf, Y = guarded(T, m, m + 8, "bf16", dev)
    dxbuf, dX = guarded(T, n, n + 24, "bf16", dev)
    c = plan_c(plan, vals, dev)
    ff.adapter_fwd(plan, Xd, c, s, Y=Y)
    Yb = ff.adapter_fwd(plan, Xd, c, s, Y=Y.clone(), beta=0.5)
    _, dC = ff.adapter_bwd(plan, Xd, Gd, c, s, dX=dX, dC=torch.full((plan.coef_slots,), float("nan"), device=dev))
    dXb, _ = ff.adapter_bwd(plan, Xd, Gd, c, s, dX=dX.clone(), beta_dx=-1.5, want_dc=False)
    _, dC2 = ff.adapter_bwd(plan, Xd, Gd, c, s, want_dx=False)
    torch.cuda.synchronize()
    assert guards_intact(ybuf, T, m, m + 8, "bf16") and guards_intact(dxbuf, T, n, n + 24, "bf16")
    P_in, P_out = oracle_frame(k_in, rn, n), oracle_frame(k_out, rm, m)
    fb = FwdBounds(P_in, P_out, rows, cols, vals, s, X[t], "bf16", k_in, k_out)
    _ok("y", to_np(Y[t]), fb.y, fb.by)
    _ok("y coef", fb.coef(to_np(Y[t])), fb.v, fb.bv)
    fbb = FwdBounds(P_in, P_out, rows, cols, vals, s, X[t], "bf16", k_in, k_out, beta_y0=0.5 * to_np(Y[t]))
    _ok("y beta", to_np(Yb[t]), fbb.y, fbb.by)
    bt = BwdBounds(P_in, P_out, rows, cols, vals, s, X[t], G[t], "bf16", k_in, k_out)
    _ok("dX", to_np(dX[t]), bt.dx, bt.bdx)
    _ok("dX coef", bt.coef(to_np(dX[t])), bt.q, bt.bq)
    bbb = BwdBounds(P_in, P_out, rows, cols, vals, s, X[t], G[t], "bf16", k_in, k_out, beta_dx0=-1.5 * to_np(dX[t]))
    _ok("dX beta", to_np(dXb[t]), bbb.dx, bbb.bdx)
    b = bt if few else BwdBounds(P_in, P_out, rows, cols, vals, s, X, G, "bf16", k_in, k_out)
    _ok("dC", user_dc(plan, dC), b.dc, b.bdc)
    assert torch.equal(dC, dC2), "dC is not deterministic"


# frames, entries, the plans' max_tokens, tokens per adapter: adapters ending in different slabs (and groups of
# blocks of different sizes, by max_tokens); several slabs per partial row (400,000 entries: 23 rows); a call
# split over the smallest pool (36 slabs of the wide side); several stages
GROUPS = [((2048, 128), (4096, 256), 20000, (400, 512, 4096, 400, 20000), (0, 5, 64, 65, 400)),
          ((2752, 16), (2048, 32), 20000, (400, 500, 9000), (400, 129, 1)),
          ((2048, 32), (2752, 16), 400000, (1700, 1700), (1700, 70)),
          ((28672, 128), (256, 16), 30000, (2400, 2500), (1300, 2400)),
          ((256, 16), (28672, 128), 30000, (2500, 2400), (2400, 1300)),
          ((1024, 2), (1024, 2), 1500, (2600, 2600, 3000), (2600, 2491, 2599))]


@pytest.mark.parametrize("ragged", [False, True], ids=["same_tokens", "per_adapter_tokens"])
@pytest.mark.parametrize("case", GROUPS, ids=lambda c: "n%d_m%d_T%d" % (c[0][0], c[1][0], max(c[4])))
def test_slab_groups(dev, case, ragged):
    """Group calls against the single calls of each plan on the adapter's own tokens.  Each is within 4.5e-3 of the
    exact result (one bf16 rounding per stage; dC: fp32 sums of rounded products), in the 2-norm."""
    (n, rn), (m, rm), nnz, max_tokens, toks = case
    T, count, s = min(max_tokens), len(toks), 0.3
    toks = toks if ragged else (T,) * count
    g = inputs.rng(n + m + nnz)
    f_in, f_out = ff.framegen(n, n // rn, rn), ff.framegen(m, m // rm, rm)
    plans = [ff.plan_create(f_in, f_out, *inputs.support(g, m, n, nnz), max_tokens=t) for t in max_tokens]
    group = ff.plan_group(plans)
    c = [plan_c(p, inputs.gaussian(g, (nnz,), std=0.02), dev) for p in plans]
    gen = torch.Generator(device=dev)
    gen.manual_seed(9)
    X, G = ([torch.randn((T, d), generator=gen, device=dev).bfloat16() for _ in plans] for d in (n, m))
    Y, dX = ([torch.full((T, d), 7.0, device=dev, dtype=torch.bfloat16) for _ in plans] for d in (m, n))
    dC = [torch.full((p.coef_slots,), float("nan"), device=dev) for p in plans]
    tokens = torch.tensor(toks, dtype=torch.int32, device=dev) if ragged else None
    ff.adapter_fwd_group(group, X, c, s, Y, tokens=tokens)
    ff.adapter_bwd_group(group, X, G, c, s, dX, dC, tokens=tokens)
    torch.cuda.synchronize()

    def close(a, b):
        d, r = (a.double() - b.double()).norm(), b.double().norm()
        return bool(d <= 9e-3 * r)

    for i, t in enumerate(toks):
        assert torch.all(Y[i][t:] == 7) and torch.all(dX[i][t:] == 7), f"adapter {i}: written past its tokens"
        y = ff.adapter_fwd(plans[i], X[i][:t], c[i], s)
        dx, dc = ff.adapter_bwd(plans[i], X[i][:t], G[i][:t], c[i], s)
        torch.cuda.synchronize()
        assert close(Y[i][:t], y) and close(dX[i][:t], dx) and close(dC[i], dc), f"adapter {i}"


@pytest.mark.parametrize("wide_in", [True, False], ids=["wide_input", "wide_output"])
def test_slab_call_split_over_workspace(dev, wide_in):
    """2400 tokens of a 28672-wide source side need more slabs than the workspace holds (36 of 64 tokens): rows
    are bitwise those of calls on the two parts."""
    wide, narrow, T = (28672, 224, 128), (256, 16, 16), 2400
    (n, ki, rn), (m, ko, rm) = (wide, narrow) if wide_in else (narrow, wide)
    g = inputs.rng(17)
    rows, cols = inputs.support(g, m, n, 30000)
    plan = ff.plan_create(ff.framegen(n, ki, rn), ff.framegen(m, ko, rm), rows, cols, max_tokens=T)
    c = plan_c(plan, inputs.gaussian(g, (30000,), std=0.02), dev)
    gen = torch.Generator(device=dev)
    gen.manual_seed(5)
    X, G = (torch.randn((T, d), generator=gen, device=dev).bfloat16() for d in (n, m))
    run = (lambda a, b: ff.adapter_fwd(plan, X[a:b], c, 0.3)) if wide_in else (
        lambda a, b: ff.adapter_bwd(plan, X[a:b], G[a:b], c, 0.3)[0])
    whole, parts = run(0, T), torch.cat([run(0, 1216), run(1216, T)])
    torch.cuda.synchronize()
    assert torch.isfinite(whole.float()).all() and torch.equal(whole, parts)


@pytest.mark.parametrize("d,rho", [(1024, 64), (640, 2)], ids=["direct", "two_stages"])
def test_slab_batch_split_over_workspace(dev, d, rho):
    """Adapters that share a plan, together more slabs than the workspace holds: bitwise the calls one by one."""
    T, count = 5120, 14
    g = inputs.rng(23)
    rows, cols = inputs.support(g, d, d, 9000)
    f = ff.framegen(d, d // rho, rho)
    plan = ff.plan_create(f, f, rows, cols, max_tokens=T, max_batch=count)
    gen = torch.Generator(device=dev)
    gen.manual_seed(6)
    X, G = (torch.randn((count, T, d), generator=gen, device=dev).bfloat16() for _ in range(2))
    c = [plan_c(plan, inputs.gaussian(g, (9000,), std=0.02), dev) for _ in range(count)]
    Y, dX = torch.zeros_like(X), torch.zeros_like(X)
    dC = [torch.empty(plan.coef_slots, device=dev) for _ in range(count)]
    ff.adapter_fwd_batched(plan, list(X), c, 0.3, list(Y))
    ff.adapter_bwd_batched(plan, list(X), list(G), c, 0.3, list(dX), dC)
    for i in range(count):
        y = ff.adapter_fwd(plan, X[i], c[i], 0.3)
        dx, dc = ff.adapter_bwd(plan, X[i], G[i], c[i], 0.3)
        torch.cuda.synchronize()
        assert torch.equal(y, Y[i]) and torch.equal(dx, dX[i]) and torch.equal(dc, dC[i])


def _bf16(x):
    return inputs.bf16_round(np.asarray(x, dtype=np.float32)).astype(np.float64)


def _factored(k):
    """The arithmetic of a factored frame's kernels, k = 4 k2: analysis and synthesis of one block.  The radix-4
    stage and its twiddles are fp32 (here float64), its results are rounded to bf16 on the way into the DFT of
    size k2, whose matrix is rounded to bf16; the synthesis rounds only its outputs."""
    k2 = k // 4
    ph = lambda x: np.exp(2j * np.pi * x)
    lb = np.outer(np.arange(k2), np.arange(k2)) % k2 / k2
    D = ph(-lb) / np.sqrt(k)
    D = _bf16(D.real) + 1j * _bf16(D.imag)
    w = np.stack([ph(a * np.arange(k2) / k) for a in range(4)])
    R = ph(np.outer(np.arange(4), np.arange(4)) / 4)

    def analysis(x):
        y = np.conj(w) * (np.conj(R) @ (x[0::2] + 1j * x[1::2]).reshape(4, k2))
        y = _bf16(y.real) + 1j * _bf16(y.imag)
        z = (y @ D.T).T.reshape(-1)          # frequency a' + 4 l
        return _bf16(np.stack([z.real, z.imag], 1).reshape(-1))

    def synthesis(z):
        y = (z[0::2] + 1j * z[1::2]).reshape(k2, 4).T @ np.conj(D)
        x = (R @ (w * y)).reshape(-1)
        return _bf16(np.stack([x.real, x.imag], 1).reshape(-1))

    return analysis, synthesis


@pytest.mark.parametrize("factored_input", [True, False], ids=["factored_input", "factored_output"])
@pytest.mark.parametrize("k", [72, 128, 172, 196, 256])
def test_factored_frames_keep_fp32_twiddles(dev, k, factored_input):
    """The results of a factored frame are those of the arithmetic above, to a few roundings that fall the other
    way (an fp32 sum of at most 512 terms is off by less than 2^-15, so about one value in 2^7 of those next to a
    rounding boundary, 2^-8 apart, moves by 2^-8: 2^-8 sqrt(2^-7) = 3.5e-4 in the 2-norm at the very most).
    Twiddles rounded to bf16 give 3e-3.  One token is not zero, so that dC is one product per entry."""
    W, kd, T, t = 2 * k, 16, 640, 37
    n, m = (W, 2 * kd) if factored_input else (2 * kd, W)
    (ki, ko) = (k, kd) if factored_input else (kd, k)
    f_in, f_out = ff.framegen(n, ki, 2), ff.framegen(m, ko, 2)
    g = inputs.rng(k)
    wide = np.arange(W)
    narrow = g.permutation(np.resize(np.arange(2 * kd), W))
    rows, cols = (narrow, wide) if factored_input else (wide, narrow)
    vals = _bf16(inputs.gaussian(g, (W,)))
    x, gr = inputs.gaussian(g, (1, n), dtype="bf16")[0], inputs.gaussian(g, (1, m), dtype="bf16")[0]
    X, G = np.zeros((T, n), np.float32), np.zeros((T, m), np.float32)
    X[t], G[t] = x, gr
    plan = ff.plan_create(f_in, f_out, rows, cols, max_tokens=T)
    Xd, Gd, c = torch_act(X, "bf16", dev), torch_act(G, "bf16", dev), plan_c(plan, vals, dev)
    dX, dC = ff.adapter_bwd(plan, Xd, Gd, c, 1.0)
    torch.cuda.synchronize()
    analysis, synthesis = _factored(k)
    P = oracle_frame(kd, 2, 2 * kd)
    B = _bf16(P.toarray() if hasattr(P, "toarray") else P)
    z = analysis(np.float64(x)) if factored_input else _bf16(B.T @ x)
    u = _bf16(B.T @ gr) if factored_input else analysis(np.float64(gr))

    def close(name, got, ref):
        err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
        assert err < 3.5e-4, f"{name}: {err:.2e} from the kernels' arithmetic"

    close("dC", user_dc(plan, dC), u[rows] * z[cols])
    if factored_input:
        close("dX", to_np(dX[t]), synthesis(_bf16(vals * u[rows])))


def test_plan_workspace_is_one_calls_scratch(dev):
    """A plan holds the scratch of one call at a time: the generic kernels' partial rows (fp32, 256 rows of the
    entry stream) and the slab kernels' slabs lie in the same memory.  A call of either kind then leaves nothing
    that the other reads."""
    n, m, T, nnz, s = 2048, 2752, 4096, 20000, 0.3
    g = inputs.rng(31)
    rows, cols = inputs.support(g, m, n, nnz)
    plan = ff.plan_create(ff.framegen(n, 64, 32), ff.framegen(m, 172, 16), rows, cols, max_tokens=T)
    slabs = (m + 1) * T * 2                                     # the wider side's coefficients
    assert plan.query(2) < slabs + 64 * 4 * 1.8 * nnz + 80 * 1.8 * nnz   # + partial rows of 64 slabs + tables
    c = plan_c(plan, inputs.gaussian(g, (nnz,), std=0.02), dev)
    gen = torch.Generator(device=dev)
    gen.manual_seed(8)
    X, G = (torch.randn((T, d), generator=gen, device=dev) for d in (n, m))
    calls = [lambda dt=dt: (ff.adapter_fwd(plan, X.to(dt), c, s), *ff.adapter_bwd(plan, X.to(dt), G.to(dt), c, s))
             for dt in (torch.float32, torch.bfloat16)]
    first = [f() for f in calls]
    again = [f() for f in calls[::-1]][::-1]
    torch.cuda.synchronize()
    for a, b in zip(first, again):
        assert all(torch.equal(x, y) for x, y in zip(a, b))
