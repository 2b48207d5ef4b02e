"""The float32 split kernel at the edges of its tiles: 16- and 32-row groups,
the 16 keys of a wave inside a 64-key unit, chunks of one unit and of several,
streams that span row groups, the self-only plan mask; against the oracle at the float32
bar (max-abs 1e-5)."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import check, dev_float, dev_int, host
from paper_2607_02963_amd import pdec

pytestmark = pytest.mark.gpu

_rng = np.random.default_rng(1)
CASES = [
    # E, L, own rows, H_q, H_kv, D, plan tokens per stream, the plan it is for: rows per group, units per chunk
    (1, 1, [1], 1, 1, 128, 0, (16, 1)),                    # one row, one prefix key
    (4, 15, [16, 17, 0, 64], 4, 1, 64, 0, (16, 1)),        # 16 rows: the one-tile group, full; wave-edge lengths
    (17, 16, [1] * 17, 1, 1, 128, 0, (32, 1)),             # 17 rows: the two-tile group
    (3, 63, [65, 15, 48], 33, 3, 128, 0, (32, 1)),         # 33 rows: a second group of one row, a stream across both
    (5, 1000, [3, 0, 40, 33, 1], 28, 4, 128, 0, (32, 1)),  # one unit per chunk
    (6, 700, [9, 9, 9, 0, 9, 9], 14, 2, 64, 20, (32, 1)),  # plan mask
    (13, 4095, [42] * 13, 28, 4, 128, 0, (32, 2)),
    # long chunks: units requested while the one before is computed, prefix and several streams' own units in one
    (40, 2000, _rng.integers(0, 100, 40).tolist(), 28, 4, 128, 0, (32, 6)),
    (24, 3000, _rng.integers(0, 70, 24).tolist(), 40, 8, 64, 0, (32, 5)),
    (16, 17000, _rng.integers(0, 70, 16).tolist(), 8, 8, 128, 0, (16, 5)),
    (40, 2000, _rng.integers(0, 100, 40).tolist(), 28, 4, 128, 10, (32, 6)),
]


@pytest.mark.parametrize("case", CASES, ids=[f"E{c[0]}L{c[1]}h{c[3]}x{c[4]}d{c[5]}p{c[6]}" for c in CASES])
def test_f32_edges_match_oracle(case):
    E, L, lens, H_q, H_kv, D, T, plan = case
    rng = np.random.default_rng(70 + E + L)
    cap = max(lens) + 1
    info = pdec.describe_plan(pdec.make_dims(E, H_q, H_kv, D, cap, L, pdec.PDEC_DTYPE_F32, plan_mask=int(T > 0), plan_per_stream=T))
    assert (info["rows_per_item"], info["chunk_keys"] // 64) == plan
    f = lambda s, *shape: (s * rng.standard_normal(shape)).astype(np.float32)  # noqa: E731
    q, kp, vp = f(1.0, E, H_q, D), f(1.0, L, H_kv, D), f(0.5, L, H_kv, D)
    ke, ve, n = f(1.0, E, cap, H_kv, D), f(0.5, E, cap, H_kv, D), np.asarray(lens, np.int32)
    out, lse = pdec.attn_step(*(dev_float(x, "f32") for x in (q, kp, vp, ke, ve)), dev_int(n), dev_int([L]),
                              plan_mask=int(T > 0), plan_per_stream=T)
    torch.cuda.synchronize()
    ref_o, ref_l = oracle.attn_step(q, kp, vp, ke, ve, n, [0, L], [0, E], **({"plan_mask": 1, "plan_per_stream": T} if T else {}))
    check("f32", host(out), host(lse), ref_o, ref_l, what=f"f32 edges {case}")
