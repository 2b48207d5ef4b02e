"""The whole-branch kernel (queries_per_stream > 1) at the edges of its tiles,
row groups, chunks and masks, against the oracle's attn_prefill.

Rows of a kv head come in waves of 32 or 64 and groups of 128 or 256; keys in
64-key units, two 32-key blocks each; a long prefix is cut into chunks merged
by the finish pass in batches of 8, 16 or 64 slots.  Each case states the row
group and the chunk it is for, which are asked for first.  The bar is the bf16 one
(P and the result are rounded to bf16): max-abs 2e-2, normwise 1e-2.
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import check, dev_float, dev_int, host
from paper_2607_02963_amd import pdec
from paper_2607_02963_amd import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [
    # E, N, L, lens, H_q, H_kv, D, cap, cross, the plan it is for: rows per group, units per chunk
    (1, 2, 1, [2], 1, 1, 128, 2, 0, (128, 2)),                      # two rows, one prefix key
    (2, 64, 31, [64, 33], 1, 1, 128, 64, 0, (128, 3)),              # 128 rows: one group, full
    (3, 43, 65, [43, 43, 1], 1, 1, 128, 70, 0, (128, 1)),           # one row in the second group; cache longer than the branch
    (1, 256, 33, [200], 1, 1, 64, 256, 0, (128, 1)),                # one stream's units, a chunk each; rows past the cache
    (1, 257, 64, [257], 1, 1, 128, 300, 0, (128, 1)),               # three groups, one row in the last
    (5, 13, 1983, [13, 0, 7, 13, 1], 14, 2, 128, 16, 0, (128, 2)),  # several chunks, a partial last prefix unit
    (9, 40, 130, [40, 64, 3, 40, 0, 40, 39, 33, 32], 4, 1, 128, 64, 1, (128, 1)),  # other streams' units, lengths above N
    (70, 2, 200, [2] * 69 + [0], 2, 2, 64, 2, 1, (128, 2)),         # more streams than one scan of the unit table
    (5, 100, 70, [100, 64, 0, 65, 3], 4, 1, 128, 100, 1, (128, 1)), # other streams' second units, which some waves see nothing of
    (3, 150, 0, [150, 129, 128], 6, 2, 64, 150, 1, (128, 1)),
    (2, 3, 9000, [3, 3], 2, 1, 128, 3, 0, (128, 1)),                # 143 slots per row
    (1, 300, 0, [300], 28, 4, 128, 300, 0, (128, 5)),               # a causal sequence: the ring refilled with own units
    (1, 300, 0, [299], 28, 4, 64, 310, 0, (128, 5)),
    (5, 64, 0, [64, 64, 0, 33, 50], 28, 4, 128, 64, 1, (128, 5)),   # one chunk of other streams' units
    (5, 64, 0, [64, 2, 64, 33, 64], 28, 4, 64, 64, 1, (128, 5)),
    # two tiles per wave
    (40, 8, 6000, [8] * 40, 28, 4, 128, 8, 0, (256, 15)),           # a last group of three full waves; few-slot rows
    (24, 37, 100, [37] * 20 + [0, 1, 36, 37], 40, 8, 128, 37, 0, (256, 5)),  # a last group that ends in a wave's second tile
    (24, 37, 100, [37] * 20 + [0, 1, 36, 37], 40, 8, 64, 37, 0, (256, 5)),
    (1, 300, 2000, [300], 28, 4, 128, 300, 0, (256, 6)),            # one stream's own units behind a prefix; 52 rows in the last group
    (1, 300, 2000, [290], 28, 4, 64, 320, 0, (256, 6)),
    (24, 10, 100, [10] * 22 + [0, 4], 40, 8, 128, 10, 1, (256, 5)), # other streams' units
    (13, 90, 0, [90] * 11 + [70, 2], 8, 8, 64, 90, 1, (256, 5)),
]


@pytest.mark.parametrize("case", CASES, ids=[f"E{c[0]}N{c[1]}L{c[2]}d{c[6]}x{c[8]}" for c in CASES])
def test_branch_edges_match_oracle(case):
    E, N, L, lens, H_q, H_kv, D, cap, cross, plan = case
    info = pdec.describe_plan(pdec.make_dims(E, H_q, H_kv, D, cap, L, pdec.PDEC_DTYPE_BF16, queries_per_stream=N,
                                             cross_causal=cross))
    assert (info["rows_per_item"], info["chunk_keys"] // 64) == plan and info["kernel_shape"] == (7 if plan[0] == 256 else 6)
    rng = np.random.default_rng(100 + E + N + L)
    f = lambda s, *shape: wl.bf16_bits((s * rng.standard_normal(shape)).astype(np.float32))  # noqa: E731
    # scores of about 1.5 nats, values that the output bar can tell apart
    q, kp, vp = f(1.5, E, N, H_q, D), f(1.0, L, H_kv, D), f(0.5, L, H_kv, D)
    ke, ve = f(1.0, E, cap, H_kv, D), f(0.5, E, cap, H_kv, D)
    n = np.asarray(lens, np.int32)
    out, lse = pdec.attn_prefill(dev_float(q, "bf16"), dev_float(kp, "bf16"), dev_float(vp, "bf16"),
                                 dev_float(ke, "bf16"), dev_float(ve, "bf16"), dev_int(n), dev_int([L]), cross=cross)
    torch.cuda.synchronize()
    ref_o, ref_l = oracle.attn_prefill(q, kp, vp, ke, ve, n, [0, L], [0, E], cross=cross)
    check("bf16", host(out).reshape(E * N, H_q, D), host(lse).reshape(E * N, H_q), ref_o.reshape(E * N, H_q, D),
          ref_l.reshape(E * N, H_q), what=f"branch edges {case}")


def test_branch_prefix_shorter_than_its_bound():
    """The plan's chunks follow the bound on the prefix; the video's prefix,
    in device memory, may be shorter, leaving slots that hold no state."""
    rng = np.random.default_rng(5)
    E, N, L, room, H_q, H_kv, D = 3, 20, 777, 5000, 14, 2, 128
    f = lambda *shape: wl.bf16_bits(rng.standard_normal(shape).astype(np.float32))  # noqa: E731
    q, kp, vp, ke, ve = f(E, N, H_q, D), f(room, H_kv, D), f(room, H_kv, D), f(E, N, H_kv, D), f(E, N, H_kv, D)
    n = np.array([20, 5, 20], np.int32)
    dims = pdec.make_dims(E, H_q, H_kv, D, N, room, pdec.PDEC_DTYPE_BF16, queries_per_stream=N)
    ws = torch.full((pdec.workspace_size(dims),), 255, dtype=torch.uint8, device="cuda")  # NaN patterns
    out, lse = pdec.attn_prefill(dev_float(q, "bf16"), dev_float(kp, "bf16"), dev_float(vp, "bf16"),
                                 dev_float(ke, "bf16"), dev_float(ve, "bf16"), dev_int(n), dev_int([L]), workspace=ws)
    torch.cuda.synchronize()
    ref_o, ref_l = oracle.attn_prefill(q, kp[:L], vp[:L], ke, ve, n, [0, L], [0, E])
    check("bf16", host(out).reshape(E * N, H_q, D), host(lse).reshape(E * N, H_q), ref_o.reshape(E * N, H_q, D),
          ref_l.reshape(E * N, H_q), what="branch short prefix")


@pytest.mark.parametrize("V,cross", [(2, 0), (5, 1), (70, 0)])
def test_branch_batch_of_unequal_videos(V, cross):
    """Videos without streams, without a prefix, with one row group and with
    several: the items that exist are numbered over the videos, 64 of them at a
    time."""
    rng = np.random.default_rng(40 + V)
    N, H_q, H_kv, D = 21, 14, 2, 128
    events = [13, 1] if V == 2 else rng.integers(0, 4, V).tolist()
    events[-1] = max(events[-1], 1)
    prefix = [1500, 900] if V == 2 else (rng.integers(0, 5, V) * 67).tolist()
    SE, SL = sum(events), sum(prefix)
    f = lambda s, *shape: wl.bf16_bits((s * rng.standard_normal(shape)).astype(np.float32))  # noqa: E731
    q, kp, vp = f(1.5, SE, N, H_q, D), f(1.0, SL, H_kv, D), f(0.5, SL, H_kv, D)
    ke, ve = f(1.0, SE, N, H_kv, D), f(0.5, SE, N, H_kv, D)
    n = rng.integers(0, N + 1, SE).astype(np.int32)
    cup, cue = np.concatenate([[0], np.cumsum(prefix)]), np.concatenate([[0], np.cumsum(events)])
    out, lse = pdec.attn_prefill_ragged(dev_float(q, "bf16"), dev_float(kp, "bf16"), dev_float(vp, "bf16"), dev_int(cup),
                                        dev_float(ke, "bf16"), dev_float(ve, "bf16"), dev_int(n), dev_int(cue),
                                        max_prefix_len=max(prefix), max_events_per_video=max(events), cross=cross)
    torch.cuda.synchronize()
    ref_o, ref_l = oracle.attn_prefill(q, kp, vp, ke, ve, n, cup.astype(np.int32), cue.astype(np.int32), cross=cross)
    check("bf16", host(out).reshape(SE * N, H_q, D), host(lse).reshape(SE * N, H_q), ref_o.reshape(SE * N, H_q, D),
          ref_l.reshape(SE * N, H_q), what=f"branch batch {V}")
