"""ff_adapter_bwd_noalloc against ff_adapter_bwd, through the C ABI.

The no-allocation backward keeps its scratch in an array of the library's code object, shared by
every call on the device and holding whatever the previous call left there.  Two calls in a row,
the second on fewer tokens (so it reads a region the first one filled with other values), must
give bitwise the results of the plain backward on the fused 128-wide kernels, the generic and the
slab ones; a call needing more scratch than the array holds is refused and writes nothing.
"""
import numpy as np
import pytest

from paper_2608_26430_amd import inputs
from tests.parity_util import torch_act

torch = pytest.importorskip("torch")
import paper_2608_26430_amd as ff  # noqa: E402
from paper_2608_26430_amd import binding  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    return torch.device("cuda:0")


def _call_pair(dev, plan, dtype, T, seed, s, beta, acc):
    n, m = plan.n, plan.m
    g = inputs.rng(seed)
    X = torch_act(inputs.gaussian(g, (T, n), dtype=dtype), dtype, dev)
    G = torch_act(inputs.gaussian(g, (T, m), dtype=dtype), dtype, dev)
    c = torch.from_numpy(plan.to_plan(inputs.gaussian(g, (plan.nnz,), std=0.02))).to(dev)
    dX0 = torch_act(inputs.gaussian(g, (T, n), dtype=dtype), dtype, dev)
    dC0 = torch.from_numpy(plan.to_plan(inputs.gaussian(g, (plan.nnz,)))).to(dev)
    ref = ff.adapter_bwd(plan, X, G, c, s, dX=dX0.clone(), dC=dC0.clone(), beta_dx=beta, accumulate_dc=acc)
    got = binding.adapter_bwd_noalloc(plan, X, G, c, s, dX0.clone(), dC0.clone(), beta_dx=beta, accumulate_dc=acc)
    # dX only and dC only (no coefficients) as well
    ref_x, _ = ff.adapter_bwd(plan, X, G, c, s, want_dc=False)
    got_x, _ = binding.adapter_bwd_noalloc(plan, X, G, c, s, torch.empty_like(ref_x), None)
    _, ref_c = ff.adapter_bwd(plan, X, G, c, s, want_dx=False)
    _, got_c = binding.adapter_bwd_noalloc(plan, X, G, None, s, None, torch.empty_like(ref_c))
    return [(ref[0], got[0]), (ref[1], got[1]), (ref_x, got_x), (ref_c, got_c)]


# (n, rho_in, m, rho_out, nnz, dtype, T first, T second): the fused 128-wide kernels at the
# q_proj layer's full 4096 tokens, the generic kernels (fp32), the slab kernels (factored blocks), and a frame in
# two stages, whose long calls run there and whose short ones run in the generic kernels
CASES = [(4096, 64, 4096, 64, 10000, "bf16", 4096, 37),
         (256, 16, 512, 32, 700, "f32", 300, 9),
         (2752, 16, 1024, 16, 4000, "bf16", 200, 3),
         (1024, 2, 1024, 2, 1500, "bf16", 2400, 70)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "n%d_m%d_%s" % (c[0], c[2], c[5]))
def test_noalloc_matches_plain_backward(dev, case):
    n, rn, m, rm, nnz, dtype, T1, T2 = case
    rows, cols = inputs.support(inputs.rng(n + m), m, n, nnz)
    f_in, f_out = ff.framegen(n, n // rn, rn), ff.framegen(m, m // rm, rm)
    plan = ff.plan_create(f_in, f_out, rows, cols, max_tokens=T1)
    first = _call_pair(dev, plan, dtype, T1, 1, 0.31, 0.0, False)
    second = _call_pair(dev, plan, dtype, T2, 2, -0.7, 0.5, True)
    torch.cuda.synchronize()
    for i, (ref, got) in enumerate(first + second):
        assert torch.equal(ref, got), f"output {i} differs from ff_adapter_bwd"


def test_noalloc_takes_uneven_supports(dev):
    """Two dense columns in each block of a 16384 x 16384 support: accepted by its 13 MiB of coefficients and
    partial sums, so it runs, however unevenly the entries lie."""
    n = 16384
    g = inputs.rng(9)
    cols = np.arange(256)
    rows = np.concatenate([g.choice(n, 6600, replace=False) for _ in cols]).astype(np.int32)
    f = ff.framegen(n, 64, 256)
    plan = ff.plan_create(f, f, rows, np.repeat(cols, 6600).astype(np.int32), max_tokens=4)
    pairs = _call_pair(dev, plan, "bf16", 4, 3, 0.2, 0.5, True)
    torch.cuda.synchronize()
    assert all(torch.equal(ref, got) for ref, got in pairs)


def test_noalloc_refuses_oversized_call(dev):
    n = m = 4096
    T = 16384
    rows, cols = inputs.support(inputs.rng(5), m, n, 10000)
    f = ff.framegen(n, 64, 64)
    plan = ff.plan_create(f, f, rows, cols, max_tokens=T)
    X = torch.zeros((T, n), dtype=torch.bfloat16, device=dev)
    G = torch.zeros((T, m), dtype=torch.bfloat16, device=dev)
    c = torch.zeros((plan.coef_slots,), device=dev)
    dX = torch.full((T, n), 3.0, dtype=torch.bfloat16, device=dev)
    dC = torch.full((plan.coef_slots,), 3.0, device=dev)
    with pytest.raises(ff.FrameFTError) as ei:
        binding.adapter_bwd_noalloc(plan, X, G, c, 1.0, dX, dC)
    assert ei.value.name == "FF_EINVAL" and "scratch" in str(ei.value)
    torch.cuda.synchronize()
    assert torch.all(dX == 3.0) and torch.all(dC == 3.0)
