"""Float calls on the matrix cores at the sizes where they can go wrong: edges of the 16-key and 16-row tiles, the waves' shares,
one run of keys and several, trees on either side of 64 nodes, sums kept aside, values and scores that are not finite."""
import numpy as np
import pytest
import torch

from paper_2502_17421_amd import binding as ls
from test_call_routes import PARENTS, Q, desc, lib, route  # noqa: F401  (lib: fixture)
from test_gpu_light_block import make
from util import DeviceBatch, gates, oracle_full

# query heads, KV heads, head_dim, tree nodes, prefix lengths, inputs
CASES = [
    (1, 1, 64, 1, [0], "iid"),                      # one row that sees one key
    (1, 1, 128, 1, [1], "iid"),
    (4, 1, 64, 4, [15, 16, 17], "peaked"),          # one tile of rows, one of keys
    (3, 1, 128, 5, [127, 128, 129, 0], "tree"),     # 15 rows; eight tiles, a wave each
    (4, 4, 64, 17, [97], "tree"),                   # 17 rows: a second tile of one
    (8, 2, 128, 8, [1000, 3], "tree"),              # 32 rows
    (8, 1, 64, 63, [300], "peaked"),
    (4, 2, 128, 64, [2049], "tree"),                # the last size masked in registers
    (4, 2, 64, 65, [2047, 511], "tree"),            # the chains are walked in LDS
    (2, 2, 128, 512, [40], "tree"),                 # the largest tree
    (16, 8, 64, 40, [4096] * 4 + [5, 4001, 0], "peaked"),  # 32 rows per workgroup, sums kept aside
    (32, 32, 128, 40, [2500, 2400], "tree"),
    (4, 1, 64, 9, [20000], "peaked"),               # the most runs
]


@pytest.mark.gpu
@pytest.mark.parametrize("hq,hkv,d,t,plens,variant", CASES)
def test_against_the_oracle(hq, hkv, d, t, plens, variant):
    batch = make("f32", hq, hkv, d, t, plens, variant, 61000 + t)
    print(f"float hq={hq} hkv={hkv} d={d} t={t} plens={plens} {variant}", flush=True)
    db = DeviceBatch(batch, token_major=t % 2 == 0)
    out, lse = db.run_full()
    torch.cuda.synchronize()
    first = out.clone(), lse.clone()
    db.workspace.fill_(0xFF)  # whatever the workspace and the outputs held, the result is the same
    out.fill_(float("nan"))
    db.run_full()
    torch.cuda.synchronize()
    assert torch.equal(out, first[0]) and torch.equal(lse, first[1])
    ro, rl = oracle_full(batch)
    print(gates(out.cpu().numpy(), lse.cpu().numpy(), ro, rl, "f32", "  whole call", stress=True), flush=True)
    # in place: the same bits where the keys are cut alike (parts of one run are divided by a sum of one weight)
    q = db.q.clone()
    at = ls.make_desc(q, db.k_cache, db.v_cache, db.k_tree, db.v_tree, q, db.desc.max_prefix_len)
    ls.ls_hybrid_tree_attn(at, q, db.k_cache, db.v_cache, db.prefix_lens, db.k_tree, db.v_tree, db.parents, q, lse, db.workspace)
    torch.cuda.synchronize()
    assert torch.equal(q, first[0])
    gates(q.cpu().numpy(), lse.cpu().numpy(), ro, rl, "f32", "  in place", stress=True)
    # cached keys only, and their pieces by the stand-alone call
    db.run_cache_only()
    torch.cuda.synchronize()
    co, cl = oracle_full(batch, use_tree=False)
    seen = np.isfinite(cl)
    got = db.lse.cpu().numpy()
    assert np.array_equal(np.isfinite(got), seen)
    gates(db.out.cpu().numpy(), np.where(seen, got, 0.0), co, np.where(seen, cl, 0.0), "f32", "  cached keys only", stress=True)
    for n in (1, 3):
        o = torch.full((len(plens), hq, n, t, d), 7.0, device="cuda")
        l = torch.full((len(plens), hq, n, t), float("nan"), device="cuda")
        ls.ls_prefix_attn_splitkv(db.desc, db.q, db.k_cache, db.v_cache, db.prefix_lens, n, o, l)
        merged, merged_lse = torch.full_like(db.out, float("nan")), torch.full_like(db.lse, float("nan"))
        ls.ls_lse_merge(ls.make_desc(db.q, db.k_cache, db.v_cache, db.k_tree, db.v_tree, merged, db.desc.max_prefix_len), n, o, l,
                        merged, merged_lse)
        torch.cuda.synchronize()
        assert torch.all(o[torch.isneginf(l)] == 7.0)  # pieces without keys leave their rows as they are
        got = merged_lse.cpu().numpy()
        assert np.array_equal(np.isfinite(got), seen)
        gates(merged.cpu().numpy(), np.where(seen, got, 0.0), co, np.where(seen, cl, 0.0), "f32", f"  {n} pieces", stress=True)


@pytest.mark.gpu
@pytest.mark.parametrize("hq,hkv,d,t,plen", [(4, 2, 128, 9, 60), (4, 1, 64, 70, 3000), (8, 2, 128, 40, 900)])
def test_what_is_not_finite_stays_with_the_rows_that_see_it(hq, hkv, d, t, plen):
    batch = make("f32", hq, hkv, d, t, [plen], "tree", 62000 + t)
    parents, node, group = batch.seqs[0].parents, t // 3, hq // hkv
    sees = np.zeros(t, bool)
    for i in range(t):
        j = i
        while j >= 0:
            sees[i] |= j == node
            j = parents[j]
    assert sees.any() and not sees.all()
    print(f"float, not finite hq={hq} hkv={hkv} d={d} t={t} plen={plen}", flush=True)

    def run():
        db.run_full()
        torch.cuda.synchronize()
        return db.out.cpu().numpy(), db.lse.cpu().numpy()

    db = DeviceBatch(batch)
    db.v_tree[:, :, node, 3] = db.v_tree[:, :, node, 40] = 0.0
    out0, lse0 = run()
    db.v_tree[:, :, node, 3] = float("-inf")
    db.v_tree[:, :, node, 40] = float("nan")
    out, lse = run()
    touched = np.zeros(out.shape, bool)
    touched[:, :, sees, 3] = touched[:, :, sees, 40] = True
    assert np.array_equal(lse, lse0) and np.array_equal(out[~touched], out0[~touched])
    assert np.all(np.isneginf(out[:, :, sees, 3])) and np.all(np.isnan(out[:, :, sees, 40]))
    # a NaN in a query row and in a cached key
    db = DeviceBatch(batch)
    ro, rl = oracle_full(batch)
    db.q[0, hq - 1, t // 2, 7] = float("nan")
    db.k_cache[0, 0, plen // 3, 5] = float("nan")
    out, lse = run()
    bad = np.zeros((1, hq, t), bool)
    bad[0, hq - 1, t // 2] = True
    bad[0, :group] = True
    assert np.isnan(lse[bad]).all() and np.isnan(out[bad]).all()
    gates(out[~bad], lse[~bad], ro[~bad], rl[~bad], "f32", "  the other rows", stress=True) if (~bad).any() else None
    # cached keys that score -inf: whole tiles at the start, a part of one, the end
    seq = batch.seqs[0]
    seq.q[..., 0] = np.abs(seq.q[..., 0]) + 2.0
    for lo, hi in ((0, 33), (plen // 2, plen // 2 + 7), (plen - 18, plen)):
        seq.k_cache[:, lo:hi, 0] = -np.inf
    db = DeviceBatch(batch)
    out, lse = run()
    ro, rl = oracle_full(batch)
    print(gates(out, lse, ro, rl, "f32", "  scores of -inf", stress=True), flush=True)


@pytest.mark.gpu
def test_sums_are_taken_in_short_runs():
    """Keys of equal weight: what is left of the error is that of the sums.  It is that of fp32 additions one by one in runs of four
    tiles of a wave, whose sums are added up in turn, then the waves' (simulated; runs of eight tiles have 1.3 times as much)."""
    b, h, d, t, plen = 8, 32, 64, 16, 4096
    rng = np.random.default_rng(64000)

    def simulated(v):  # [keys, columns]
        tiles = v.reshape(-1, 4, 4, v.shape[1]).transpose(0, 2, 1, 3).reshape(-1, 16, v.shape[1])  # in the order of the products
        total = np.zeros(v.shape[1], np.float32)
        for wave in range(8):
            kept = run = np.zeros(v.shape[1], np.float32)
            for i, tile in enumerate(tiles[wave::8]):
                for row in tile:
                    run = run + row
                if i % 4 == 3:
                    kept, run = kept + run, np.zeros_like(run)
            total = total + (kept + run)
        return total / np.float32(len(v))

    rel = lambda x, ref: float(np.sqrt(np.mean((x - ref) ** 2) / np.mean(ref ** 2)))
    sample = rng.standard_normal((plen, 4096), dtype=np.float32)
    expect = rel(simulated(sample).astype(np.float64), sample.astype(np.float64).mean(0))
    q, k = torch.zeros((b, h, t, d), device="cuda"), torch.zeros((b, h, plen, d), device="cuda")
    v = torch.from_numpy(rng.standard_normal((b, h, plen, d), dtype=np.float32)).cuda()
    out, lse = torch.zeros_like(q), torch.zeros((b, h, t), device="cuda")
    x = ls.make_desc(q, k, v, q, q, out, plen)
    print("float, equal weights", flush=True)
    ls.ls_cache_attn(x, q, k, v, torch.full((b,), plen, dtype=torch.int32, device="cuda"), out, lse,
                     torch.empty(ls.ls_workspace_bytes(x), dtype=torch.uint8, device="cuda"))
    ref = v.double().mean(2, keepdim=True).expand(-1, -1, t, -1)
    got = rel(out.double().cpu().numpy(), ref.cpu().numpy())
    print(f"  {got:.3e}, simulated {expect:.3e}", flush=True)
    assert got <= 1.1 * expect


@pytest.mark.gpu
def test_bad_parents_are_cut_and_reported():
    for t, plen in ((40, 100), (100, 2000)):
        batch = make("f32", 4, 2, 64, t, [plen, plen], "tree", 63000 + t)
        db = DeviceBatch(batch)
        bad = np.stack([s.parents for s in batch.seqs])
        bad[1][t // 2], bad[1][t - 1] = t - 1, -7
        cut = bad.copy()
        cut[1][t // 2], cut[1][t - 1] = -1, -1
        results = []
        for parents in (bad, cut):
            db.parents = torch.from_numpy(parents).cuda()
            db.run_full()
            torch.cuda.synchronize()
            at = ls.ls_workspace_error(db.desc, db.workspace) - db.workspace.data_ptr()
            results.append((db.out.clone(), db.lse.clone(), db.workspace[at:at + 8].view(torch.int32).cpu().tolist()))
        assert results[0][2] == [0, 1] and results[1][2] == [0, 0]
        assert torch.equal(results[0][0], results[1][0]) and torch.equal(results[0][1], results[1][1])


def test_routes(lib):
    """One launch while the keys are few; runs of keys and a merge, of one run too where the outputs lie over inputs.  The workspace
    holds the parts of ls_prefix_num_splits runs, so there are never more.  (The stand-in prints 32 rows for a tile of 16.)"""
    call = lambda *sizes, **at: route(lib, desc(*sizes, dtype=ls.LS_F32), **at)
    assert call(4, 1, 64, 16, 100) == ["wave_split(rows=32,splits=1,tree)"]
    assert call(4, 1, 64, 16, 100, out=Q) == ["wave_split(rows=32,splits=1,tree)", "merge"]
    assert call(4, 1, 64, 16, 100, lse=PARENTS) == ["wave_split(rows=32,splits=1,tree)", "merge"]
    assert call(4, 1, 64, 16, 1024) == ["wave_split(rows=32,splits=16,tree)", "merge"]
    assert call(4, 1, 64, 16, 1024, tree=False) == ["wave_split(rows=32,splits=16)", "merge"]
    for sizes in ((4, 1, 64, 1, 0), (32, 8, 128, 40, 4096, 8), (8, 2, 128, 512, 2 ** 31 - 1), (64, 64, 64, 4, 70, 1000)):
        x = desc(*sizes, dtype=ls.LS_F32)
        most = ls.ls_prefix_num_splits(x)
        for tree in (True, False):
            first = route(lib, x, tree=tree)
            n = int(first[0].split("splits=")[1].rstrip(")").split(",")[0])
            assert first[0].startswith("wave_split(") and 1 <= n <= most and len(first) == (1 if n == 1 else 2)


def test_large_trees_are_counted_as_the_last_run_takes_them(lib):
    """All tree tiles go to the last run of keys, so more runs than leave it with an equal share make nothing shorter."""
    for sizes in ((2, 2, 128, 512, 1000), (2, 2, 128, 512, 2000), (2, 2, 128, 300, 700), (1, 1, 64, 512, 3000)):
        first = route(lib, desc(*sizes, dtype=ls.LS_F32))[0]
        n = int(first.split("splits=")[1].rstrip(")").split(",")[0])
        tree_tiles, tiles = (sizes[3] + 15) // 16, (sizes[4] + 15) // 16 + (sizes[3] + 15) // 16
        assert n > 1 and -(-tiles // (n - 1)) > tree_tiles, (sizes, n)  # (one run fewer would be longer than the tree)
