"""The cached-key kernel with blocks of 128 query rows, whose other four waves copy, at the sizes where it can go wrong:
edges of blocks and of waves, odd tile counts, both windows, pages, tree keys on the last split.  Its parts are those of
the blocks of 256 rows bit for bit: a wave does the same whoever copies for it."""
import sys

import numpy as np
import pytest
import torch

from paper_2502_17421_amd import binding as ls
from test_gpu_light_block import make
from test_gpu_paged import PagedBatch
from util import DeviceBatch, gates, oracle_full

pytestmark = pytest.mark.gpu

# dtype, query heads, KV heads, head_dim, tree nodes, prefix lengths, inputs
CASES = [
    ("bf16", 8, 2, 128, 64, [4400], "peaked"),       # 256 rows: two whole blocks, short splits
    ("f16", 8, 2, 128, 33, [5000], "tree"),          # 132 rows: the second block has four
    ("bf16", 4, 2, 64, 65, [4500], "peaked"),        # 130 rows
    ("f16", 6, 2, 128, 43, [4711], "tree"),          # 129 rows
    ("bf16", 8, 4, 128, 150, [4403], "tree"),        # 300 rows: three blocks, the last one of 44
    ("bf16", 2, 2, 128, 128, [9001], "peaked"),      # 128 rows
    ("f16", 5, 1, 128, 13, [40000], "tree"),         # 65 rows, long splits, tree keys on the last one
    ("bf16", 8, 2, 64, 24, [30011, 900], "tree"),    # 96 rows, pieces dealt by length
]


@pytest.mark.parametrize("dtype,hq,hkv,d,t,plens,variant", CASES)
def test_whole_call_against_the_oracle(dtype, hq, hkv, d, t, plens, variant):
    batch = make(dtype, hq, hkv, d, t, plens, variant, 51000 + t)
    print(f"row blocks {dtype} hq={hq} hkv={hkv} d={d} t={t} plens={plens} {variant}", flush=True)
    db = DeviceBatch(batch, token_major=t % 2 == 0)
    out, lse = db.run_full()
    torch.cuda.synchronize()
    ro, rl = oracle_full(batch)
    print(gates(out.float().cpu().numpy(), lse.cpu().numpy(), ro, rl, dtype, "  result", stress=True), flush=True)
    pb = PagedBatch(batch, 16 if t % 3 else 64, np.random.default_rng(5))
    po, pl = pb.run()
    if pb.desc.max_prefix_len == db.desc.max_prefix_len:
        assert np.array_equal(po, out.float().cpu().numpy()) and np.array_equal(pl, lse.cpu().numpy())


@pytest.mark.parametrize("dtype,hq,hkv,d,t,plen,n_splits", [
    ("bf16", 8, 2, 128, 64, 1000, 4),    # short splits
    ("bf16", 8, 2, 128, 64, 3333, 3),    # long ones
    ("f16", 8, 2, 64, 40, 2010, 5),
    ("bf16", 6, 2, 128, 43, 31, 1),      # one tile
    ("f16", 4, 2, 128, 130, 700, 2),     # 260 rows
])
def test_parts_do_not_depend_on_the_block(dtype, hq, hkv, d, t, plen, n_splits):
    """One sequence takes blocks of 128 rows, so many copies of it that all blocks fill the chip take blocks of 256."""
    copies = 256 // (hkv * n_splits) + 1
    one = make(dtype, hq, hkv, d, t, [plen], "peaked", 52000 + t)
    many = make(dtype, hq, hkv, d, t, [plen] * copies, "peaked", 52000 + t)
    for seq in many.seqs:
        seq.q, seq.k_cache, seq.v_cache = one.seqs[0].q, one.seqs[0].k_cache, one.seqs[0].v_cache
    assert 3 * hkv * n_splits <= 256
    print(f"blocks {dtype} hq={hq} hkv={hkv} d={d} t={t} plen={plen} splits={n_splits}", flush=True)
    got = []
    for batch in (one, many):
        db = DeviceBatch(batch)
        o = torch.full((len(batch.seqs), hq, n_splits, t, d), float("nan"), device="cuda")
        lse = torch.full((len(batch.seqs), hq, n_splits, t), float("nan"), device="cuda")
        ls.ls_prefix_attn_splitkv(db.desc, db.q, db.k_cache, db.v_cache, db.prefix_lens, n_splits, o, lse)
        torch.cuda.synchronize()
        got.append((o, lse))
    sys.stdout.flush()
    filled = torch.isfinite(got[0][1][0])
    assert filled.any()
    for b in (0, copies // 2, copies - 1):
        assert torch.equal(got[0][1][0], got[1][1][b])
        assert torch.equal(got[0][0][0][filled], got[1][0][b][filled])


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,hq,hkv,d,t,plen,n_splits", [
    ("bf16", 4, 2, 64, 24, 700, 2),      # 48 rows
    ("f16", 4, 2, 64, 64, 3333, 3),      # 128 rows
])
def test_parts_do_not_depend_on_the_copying_waves(dtype, hq, hkv, d, t, plen, n_splits):
    """At head_dim 64 one sequence takes blocks with waves that copy; of so many copies of it that all blocks fill the chip the
    blocks' waves copy for themselves."""
    test_parts_do_not_depend_on_the_block(dtype, hq, hkv, d, t, plen, n_splits)
