"""Infinities and NaN stay where the mask lets them go.

A masked key has probability 0, but 0 times an infinite or NaN value is NaN, so
a work-group that multiplies a value row for some of its query rows can spoil
the others.  The runs below differ from a finite run in one place; the outputs
that do not see that place have to keep their bits.  And a live row whose
<dO, O> overflows is a live row: its gradient shows it.
"""
import numpy as np
import pytest
import torch

import backward
import oracle
from gpu_util import dev_float, dev_int
from paper_2607_02963_amd import pdec
from paper_2607_02963_amd import workloads as wl

pytestmark = pytest.mark.gpu


VALUES = [float("nan"), float("inf")]


def _normal(seed, shape, sigma=1.0, dtype=torch.bfloat16):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return (torch.randn(shape, generator=g, device="cuda") * sigma).to(dtype)


def _same(a, b):
    return torch.equal(a, b) and bool(torch.isfinite(b).all())


@pytest.mark.parametrize("bad", VALUES)
@pytest.mark.parametrize("E,N,L,H_q,H_kv,D,cross", [
    (1, 200, 0, 1, 1, 128, 0),    # one stream, one head: a group spans several units
    (1, 700, 70, 7, 1, 64, 0),
    (1, 2300, 0, 14, 2, 128, 0),  # 256-row groups
    (5, 13, 300, 28, 4, 128, 0),  # several streams in a group and in a wave
    (9, 40, 130, 4, 1, 128, 1),   # the causal-attention variant
    (3, 100, 4000, 40, 8, 64, 0),
])
def test_a_branch_value_reaches_only_rows_that_may_see_its_block(E, N, L, H_q, H_kv, D, cross, bad):
    q, kp, vp = _normal(1, (E, N, H_q, D)), _normal(2, (L, H_kv, D)), _normal(3, (L, H_kv, D), 0.5)
    ke, ve = _normal(4, (E, N, H_kv, D)), _normal(5, (E, N, H_kv, D), 0.5)
    n, plen = dev_int([N] * E), dev_int([L])
    call = lambda v: pdec.attn_prefill(q, kp, vp, ke, v, n, plen, cross=cross)  # noqa: E731
    out, lse = call(ve)
    e, t = E // 2, N - 2
    ve2 = ve.clone()
    ve2[e, t] = bad
    out2, lse2 = call(ve2)
    torch.cuda.synchronize()
    assert torch.equal(lse, lse2)  # values have no part in it
    assert not torch.isfinite(out2[e, t:]).any()
    block = 32 * (t // 32)  # rows see a 32-key block whole or in part, or not at all
    assert _same(out[e, :block], out2[e, :block])
    for f in range(E):
        if f != e:
            upto = block if cross else N
            assert _same(out[f, :upto], out2[f, :upto]), f


@pytest.mark.parametrize("bad", VALUES)
@pytest.mark.parametrize("E,N,L,H_q,H_kv,D", [(2, 40, 100, 7, 1, 128), (1, 2300, 0, 14, 2, 128), (24, 80, 700, 40, 8, 64)])
def test_a_query_row_reaches_its_own_result_only(E, N, L, H_q, H_kv, D, bad):
    q, kp, vp = _normal(1, (E, N, H_q, D)), _normal(2, (L, H_kv, D)), _normal(3, (L, H_kv, D), 0.5)
    ke, ve, n, plen = _normal(4, (E, N, H_kv, D)), _normal(5, (E, N, H_kv, D), 0.5), dev_int([N] * E), dev_int([L])
    out, lse = pdec.attn_prefill(q, kp, vp, ke, ve, n, plen)
    q2 = q.clone()
    hit = torch.zeros((E, N, H_q), dtype=torch.bool, device="cuda")
    for e, j, h in ((0, 0, 0), (E - 1, N // 2, H_q - 1), (E // 2, N - 1, H_q // 2)):
        hit[e, j, h] = True
        q2[e, j, h, 5] = bad
    out2, lse2 = pdec.attn_prefill(q2, kp, vp, ke, ve, n, plen)
    torch.cuda.synchronize()
    assert not torch.isfinite(out2[hit]).any()
    assert _same(out[~hit], out2[~hit]) and _same(lse[~hit], lse2[~hit])


@pytest.mark.parametrize("bad", VALUES)
@pytest.mark.parametrize("E,L,H_q,H_kv,D,plan", [(8, 300, 4, 1, 128, 0), (5, 130, 28, 4, 64, 0), (48, 8000, 4, 2, 128, 0),
                                                  (8, 256, 4, 1, 128, 16)])
def test_a_float32_stream_value_reaches_its_own_rows_only(E, L, H_q, H_kv, D, plan, bad):
    f32 = torch.float32
    q, kp, vp = _normal(1, (E, H_q, D), 1.0, f32), _normal(2, (L, H_kv, D), 1.0, f32), _normal(3, (L, H_kv, D), 0.5, f32)
    ke, ve = _normal(4, (E, 20, H_kv, D), 1.0, f32), _normal(5, (E, 20, H_kv, D), 0.5, f32)
    n, plen = dev_int([9 + e % 11 for e in range(E)]), dev_int([L])
    call = lambda v, p: pdec.attn_step(q, kp, p, ke, v, n, plen, plan_mask=int(plan > 0), plan_per_stream=plan)  # noqa: E731
    out, lse = call(ve, vp)
    e = E // 2
    ve2, vp2 = ve.clone(), vp.clone()
    if plan:
        vp2[L - E * plan + e * plan + 3] = bad  # one of stream e's own plan tokens
    else:
        ve2[e, 4] = bad
    out2, lse2 = call(ve2, vp2)
    torch.cuda.synchronize()
    assert torch.equal(lse, lse2)
    assert not torch.isfinite(out2[e]).any()
    for f in range(E):
        if f != e:
            assert _same(out[f], out2[f]), f


@pytest.mark.parametrize("bad", VALUES)
def test_a_row_gradient_reaches_only_key_units_it_may_see(bad):
    """dO of an early token is not finite: the cache rows of later 64-key units, which it does not see, keep their
    gradients (a 128-key tile walks the rows of both of its units)."""
    N, H, D = 192, 2, 128
    q, do = _normal(1, (1, N, H, D)), _normal(2, (1, N, H, D), 0.5)
    kp = vp = torch.empty((0, H, D), dtype=torch.bfloat16, device="cuda")
    ke, ve, n, plen = _normal(3, (1, N, H, D)), _normal(4, (1, N, H, D), 0.5), dev_int([N]), dev_int([0])
    out, lse = pdec.attn_prefill(q, kp, vp, ke, ve, n, plen)
    do2 = do.clone()
    do2[0, 10] = bad
    a = pdec.attn_prefill_backward(q, kp, vp, ke, ve, n, plen, out, lse, do)
    b = pdec.attn_prefill_backward(q, kp, vp, ke, ve, n, plen, out, lse, do2)
    torch.cuda.synchronize()
    assert not torch.isfinite(b[0][0, 10]).any() and _same(a[0][0, 11:], b[0][0, 11:]) and _same(a[0][0, :10], b[0][0, :10])
    for g in (3, 4):
        assert not torch.isfinite(b[g][0, :11]).any()
        assert _same(a[g][0, 64:], b[g][0, 64:])


@pytest.mark.parametrize("E,N,L,lens,H_q,H_kv,D", [
    (3, 40, 300, [40, 0, 33], 4, 2, 128),
    (5, 52, 257, [52, 3, 52, 52, 0], 5, 1, 128),   # many rows over few keys
    (2, 5, 4000, [5, 4], 6, 2, 64),                # few rows over many keys
    (1, 129, 0, [129], 7, 1, 128),                 # a causal sequence
])
def test_a_live_row_whose_output_product_overflows_stays_live(E, N, L, lens, H_q, H_kv, D):
    """<dO, O> = +inf in one row: its p dO reaches dv, which stays finite and right, and its ds makes dk show it."""
    rng = np.random.default_rng(17 + N)
    f = lambda s, *shape: wl.bf16_bits((s * rng.standard_normal(shape)).astype(np.float32))  # noqa: E731
    q, kp, vp = f(1.0, E, N, H_q, D), f(1.0, L, H_kv, D), f(0.5, L, H_kv, D)
    ke, ve, do = f(1.0, E, N, H_kv, D), f(0.5, E, N, H_kv, D), f(0.5, E, N, H_q, D)
    n = np.asarray(lens, np.int32)
    out, lse = oracle.attn_prefill(q, kp, vp, ke, ve, n, [0, L], [0, E])
    out_b, lse_f = wl.bf16_bits(out.astype(np.float32)), lse.astype(np.float32)
    j = 3
    out_b[0, j, 0, 0] = wl.bf16_bits(np.asarray([4.0], np.float32))[0]
    do[0, j, 0, 0] = wl.bf16_bits(np.asarray([2.0e38], np.float32))[0]  # 8e38: past the largest float32
    d = [dev_float(x, "bf16") for x in (q, kp, vp, ke, ve)]
    g = pdec.attn_prefill_backward(*d, dev_int(n), dev_int([L]), dev_float(out_b, "bf16"),
                                   torch.from_numpy(np.ascontiguousarray(lse_f)).cuda(), dev_float(do, "bf16"))
    torch.cuda.synchronize()
    ref = backward.attn_prefill_backward(q, kp, vp, ke, ve, n, out_b, lse_f, do)
    for i, name in ((2, "dv_prefix"), (4, "dv_event")):
        got, r = g[i].cpu().numpy().astype(np.float64), np.asarray(ref[i], np.float64).reshape(g[i].shape)
        assert np.isfinite(got).all(), name
        # p is rounded to bf16: 2^-9 relative in the one term that rules the norm, at most 2^-8
        assert np.linalg.norm(got - r) <= 1e-2 * np.linalg.norm(r) + 1e-12, name
    assert not torch.isfinite(g[0][0, j, 0]).any()
    if L:
        assert not torch.isfinite(g[1][:, 0]).any()
        assert torch.isfinite(g[1][:, 1:]).all()
    assert not torch.isfinite(g[3][0, :min(j + 1, lens[0]), 0]).any()
