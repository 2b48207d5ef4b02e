"""The backward's tiles, splits and masks at their edges, against the oracle's
gradients: 128-key tiles and 64-row stages of dk, dv, 256-row groups and
64-key units of dq, row splits and key splits, the small tiles (64 keys, 64
rows), ended streams, caches longer than a branch, prefixes shorter than their
bound.  Each case states the plan it is for, which is asked for first.

The bar is normwise: p and ds are rounded to bf16 (2^-9 relative, random), so
a gradient's relative error stays near 2e-3; 1e-2 leaves room for sums that
cancel.  Rows no query sees, and
ended streams' rows, are exactly zero.
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

CASES = [
    # E, N, L, room, lens, H_q, H_kv, D, cap, plan: tiles, row splits above 1, key splits above 1
    (1, 1, 1, 1, [1], 1, 1, 128, 1, "small"),                        # one row, one prefix key, one own key
    (1, 129, 0, 0, [129], 7, 1, 128, 129, "large rows"),             # pure causal, a key past one tile
    (2, 200, 0, 0, [200, 150], 4, 1, 64, 260, "large"),              # caches longer than the branch; two streams
    (3, 64, 128, 128, [64, 0, 64], 4, 4, 128, 64, "small"),          # 192 rows: full tiles, an ended stream
    (5, 52, 257, 300, [52, 3, 52, 52, 0], 5, 1, 128, 64, "large rows"),    # many rows over few keys; a short prefix
    (2, 5, 4000, 4100, [5, 4], 6, 2, 128, 5, "large keys"),          # few rows over many keys
    (7, 9, 1000, 1000, [9, 9, 0, 9, 1, 9, 9], 3, 3, 64, 9, "large keys"),  # several streams in a row group
    (2, 40, 128, 128, [40, 33], 7, 1, 128, 40, "large"),             # 280 rows and a prefix, unsplit; two row groups
    (5, 64, 128, 130, [64, 0, 63, 1, 64], 4, 2, 128, 70, "small"),         # two keys past a tile that hold nothing
    (4, 30, 130, 200, [30, 0, 17, 30], 6, 6, 64, 40, "small"),       # D = 64; a prefix past two units; caches longer
    (9, 11, 320, 320, [11, 11, 3, 0, 11, 11, 11, 1, 11], 28, 4, 128, 11, "small"),  # several streams in a row tile
]


def _plan(E, N, room, H_q, H_kv, D, cap):
    small, rows, keys = pdec.query_backward_plan(
        pdec.make_dims(E, H_q, H_kv, D, cap, room, pdec.PDEC_DTYPE_BF16, queries_per_stream=N))
    return ("small" if small else "large") + (" rows" if rows > 1 else "") + (" keys" if keys > 1 else "")


@pytest.mark.parametrize("case", CASES, ids=[f"E{c[0]}N{c[1]}L{c[2]}d{c[7]}" for c in CASES])
def test_backward_edges_match_oracle(case):
    E, N, L, room, lens, H_q, H_kv, D, cap, plan = case
    assert _plan(E, N, room, H_q, H_kv, D, cap) == plan
    rng = np.random.default_rng(300 + E + N + L)
    f = lambda s, *shape: wl.bf16_bits((s * rng.standard_normal(shape)).astype(np.float32))  # noqa: E731
    q, kp, vp = f(1.2, E, N, H_q, D), f(1.0, room, H_kv, D), f(0.5, room, H_kv, D)
    ke, ve, do = f(1.0, E, cap, H_kv, D), f(0.5, E, cap, H_kv, D), f(0.5, E, N, H_q, D)
    n = np.asarray(lens, np.int32)
    out, lse = oracle.attn_prefill(q, kp[:L], vp[:L], ke, ve, n, [0, L], [0, E])
    out_b, lse_f = wl.bf16_bits(out.astype(np.float32)), lse.astype(np.float32)
    d = [dev_float(x, "bf16") for x in (q, kp, vp, ke, ve)]
    args = (*d, dev_int(n), dev_int([L]), dev_float(out_b, "bf16"), torch.from_numpy(np.ascontiguousarray(lse_f)).cuda(),
            dev_float(do, "bf16"))
    grads = pdec.attn_prefill_backward(*args)
    again = pdec.attn_prefill_backward(*args)
    torch.cuda.synchronize()
    ref = backward.attn_prefill_backward(q, kp[:L], vp[:L], ke, ve, n, out_b, lse_f, do)
    for name, g, g2, r in zip(("dq", "dkp", "dvp", "dke", "dve"), grads, again, ref):
        assert torch.equal(g, g2), name
        got = g.cpu().numpy().astype(np.float64)
        if name in ("dkp", "dvp"):
            assert np.all(got[L:] == 0.0), name  # rows past the prefix are written, as zeros
            got = got[:L]
        if not got.size:
            continue
        r = np.asarray(r, np.float64).reshape(got.shape)
        assert np.linalg.norm(got - r) <= 1e-2 * np.linalg.norm(r) + 1e-12, (name, case)
    for e, ne in enumerate(lens):
        assert torch.all(grads[3][e, ne:] == 0) and torch.all(grads[4][e, ne:] == 0)
        if ne == 0:
            assert torch.all(grads[0][e] == 0)
