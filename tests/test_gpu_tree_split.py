"""Tree keys on the last key split of the cached-key kernel (more than 64 query rows per KV head, splits of
768 rows or more, trees of at most 256 nodes; test_call_routes.py says which call takes which kernels),
at the sizes where it can go wrong: one and several rounds of three tree tiles,
trees on both sides of the 64 nodes whose mask is built in registers, workgroups of four and eight
waves, a last row block without rows in some waves, sequences of unlike length (whose splits are dealt by
length, up to 32 sequences) with few tiles or none,
and values that must not reach rows that do not see them."""
import numpy as np
import pytest
import torch

from paper_2502_17421_amd import binding as ls
from paper_2502_17421_amd import synth
from test_gpu_light_block import make
from test_gpu_paged import PagedBatch
from util import DeviceBatch, gates, oracle_full

# dtype, query heads, KV heads, head_dim, tree nodes, prefix lengths, inputs
CASES = [
    ("bf16", 40, 8, 128, 17, [3200] + [40, 1000, 0] * 2 + [3101], "peaked"),   # 85 rows: four waves, one tree tile
    ("f16", 64, 16, 64, 32, [3200, 0, 31, 2500], "tree"),       # 128 rows; a sequence without cached keys
    ("bf16", 32, 8, 128, 64, [6300, 1700, 900, 6200], "tree"),  # the last size masked in registers; eight waves
    ("bf16", 32, 8, 64, 65, [6300, 6000], "peaked"),            # 65: the chains are walked in LDS; 260 rows
    ("f16", 32, 8, 128, 69, [12345], "tree"),                   # 276 rows, three tree tiles
    ("bf16", 32, 32, 128, 97, [4001, 33], "tree"),              # four tree tiles: a second round
    ("f16", 16, 16, 64, 128, [4000, 300, 0], "peaked"),         # 128 rows, four waves, two rounds
    ("f16", 32, 16, 64, 130, [3200, 300], "peaked"),
    ("bf16", 32, 16, 64, 200, [3300, 800], "tree"),             # seven tree tiles: three rounds
    ("bf16", 8, 8, 128, 256, [12000, 10], "tree"),              # the largest tree that rides, eight tiles
    ("bf16", 8, 4, 64, 40, [2000] * 3 + [0, 1, 31, 32, 33, 700, 1999] + [1600] * 22, "tree"),  # 32 sequences: the most
    ("bf16", 4, 2, 64, 40, [2500] * 3 + [0, 1, 31, 32, 33, 700, 1999] + [1600] * 23, "tree"),  # 33: an even cut of each
]
# the same lengths of splits, but the tail kernel takes the tree keys: more than eight tree tiles
ON_THE_TAIL = [
    ("f16", 8, 8, 128, 257, [6500, 10], "tree"),
    ("bf16", 8, 8, 128, 512, [6500, 10], "tree"),               # the largest tree, sixteen tiles
]


def whole_call(db):
    out, lse = db.run_full()
    torch.cuda.synchronize()
    return out.float().cpu().numpy(), lse.cpu().numpy()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,hq,hkv,d,t,plens,variant", CASES + ON_THE_TAIL)
def test_whole_call_against_the_oracle_and_the_tail_kernel(dtype, hq, hkv, d, t, plens, variant):
    batch = make(dtype, hq, hkv, d, t, plens, variant, 31000 + t)
    print(f"tree split {dtype} hq={hq} hkv={hkv} d={d} t={t} plens={plens} {variant}", flush=True)
    db = DeviceBatch(batch, token_major=t % 2 == 0)
    assert ls.ls_prefix_num_splits(db.desc) > 1 or len(plens) == 1
    if len(plens) < 33:
        assert ls.ls_prefix_split_len(db.desc, 0) >= 768
    first = whole_call(db)
    db.workspace.fill_(0xFF)  # whatever the workspace and the outputs held, the result is the same
    db.out.fill_(float("nan"))
    out, lse = whole_call(db)
    assert np.array_equal(out, first[0]) and np.array_equal(lse, first[1])
    ro, rl = oracle_full(batch)
    print(gates(out, lse, ro, rl, dtype, "  tree split", stress=True), flush=True)
    # in place (q is the output): the tail kernel takes the tree keys
    q = db.q.clone()
    db.workspace.fill_(0xFF)
    ls.ls_hybrid_tree_attn(ls.make_desc(q, db.k_cache, db.v_cache, db.k_tree, db.v_tree, q, db.desc.max_prefix_len), q,
                           db.k_cache, db.v_cache, db.prefix_lens, db.k_tree, db.v_tree, db.parents, q, db.lse, db.workspace)
    torch.cuda.synchronize()
    print(gates(q.float().cpu().numpy(), db.lse.cpu().numpy(), ro, rl, dtype, "  in place", stress=True), flush=True)
    # cached keys only
    db.run_cache_only()
    torch.cuda.synchronize()
    co, cl = oracle_full(batch, use_tree=False)
    seen = np.isfinite(cl)
    got = db.lse.cpu().numpy()
    assert np.array_equal(np.isfinite(got), seen)
    print(gates(db.out.float().cpu().numpy(), np.where(seen, got, 0.0), co, np.where(seen, cl, 0.0), dtype,
                "  cached keys only", stress=True), flush=True)
    # the same cache in shuffled pages
    pb = PagedBatch(batch, 16 if t % 3 else 64, np.random.default_rng(5))
    po, pl = pb.run()
    if pb.desc.max_prefix_len == db.desc.max_prefix_len:  # the same plan: bit for bit
        assert np.array_equal(po, out) and np.array_equal(pl, lse)
    print(gates(po, pl, ro, rl, dtype, "  paged", stress=True), flush=True)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,hq,hkv,d,t,plen", [("bf16", 32, 8, 128, 40, 24000), ("f16", 32, 32, 64, 100, 6500),
                                                    ("bf16", 4, 2, 128, 9, 200), ("f16", 4, 4, 64, 70, 100)])
def test_infinite_values_stay_with_the_rows_that_see_them(dtype, hq, hkv, d, t, plen):
    """A node with an infinite and a NaN value: its descendants' two columns are not finite, everything else
    is what it is with zeros there (on the kernel whose waves split the keys too)."""
    batch = make(dtype, hq, hkv, d, t, [plen], "tree", 32000 + t)
    parents = batch.seqs[0].parents
    node = t // 3
    sees = np.zeros(t, bool)
    for i in range(t):
        j = i
        while j >= 0:
            sees[i] |= j == node
            j = parents[j]
    assert sees.any() and not sees.all()
    print(f"infinite values {dtype} d={d} t={t} plen={plen}", flush=True)
    db = DeviceBatch(batch)
    db.v_tree[:, :, node, 3] = 0.0
    db.v_tree[:, :, node, 40] = 0.0
    out0, lse0 = whole_call(db)
    db.v_tree[:, :, node, 3] = float("-inf")
    db.v_tree[:, :, node, 40] = float("nan")
    out, lse = whole_call(db)
    assert np.array_equal(lse, lse0)
    touched = np.zeros(out.shape, bool)
    touched[:, :, sees, 3] = touched[:, :, sees, 40] = True
    assert np.array_equal(out[~touched], out0[~touched])
    assert np.all(np.isneginf(out[:, :, sees, 3])) and np.all(np.isnan(out[:, :, sees, 40]))


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,hq,hkv,d,t,plen", [("f16", 64, 32, 64, 40, 7000), ("f16", 32, 8, 128, 64, 26000),
                                                    ("f16", 32, 8, 128, 16, 9000), ("bf16", 32, 8, 128, 64, 26000)])
@pytest.mark.parametrize("gap", [22.7, 90.0])
def test_cached_keys_far_below_the_tree_keep_their_bits(dtype, hq, hkv, d, t, plen, gap):
    """Every cached key scores 2^-gap of every node, the nodes' values are zero: what is left in the output is the
    cached keys' part, with the relative error of any other output.  (16 nodes: the kernel whose waves split
    the keys.)  All scores are exact and equal, so numerators are powers of two next to their own reference;
    what remains is the rounding of the parts and of the output, one half-ulp each, and the fp32 sums.
    At 2^-90 the output is zero."""
    batch = make(dtype, hq, hkv, d, t, [plen], "iid", 34000 + t)
    seq = batch.seqs[0]
    seq.q[...] = 0.0
    seq.q[..., 0] = 4.0
    seq.k_cache[..., 0] = 0.0
    seq.k_tree[..., 0] = synth.round_to(np.float32(gap * np.log(2) * np.sqrt(d) / 4), dtype)
    seq.v_tree[...] = 0.0
    seq.v_cache[...] = synth.round_to(np.abs(seq.v_cache) + 0.5, dtype)
    print(f"far below {dtype} hq={hq} hkv={hkv} d={d} t={t} plen={plen} 2^-{gap}", flush=True)
    db = DeviceBatch(batch)
    out, lse = whole_call(db)
    ro, rl = oracle_full(batch)
    assert np.abs(lse - rl).max() <= 1e-5 * np.abs(rl).max()
    half_ulp = 2.0 ** -11 if dtype == "f16" else 2.0 ** -8  # of 11 and 8 significant bits, relative
    if gap > 64:
        assert np.abs(out - ro).max() <= 2.0 ** -25
    else:
        worst = (np.abs(out - ro) / ro).max()
        print(f"  relative error {worst:.2e}, half an ulp {half_ulp:.2e}", flush=True)
        assert worst <= 2.2 * half_ulp


def half_spacing(a, b, dtype):
    """Half the distance between neighbouring values of the type at |a| or |b|, the larger one."""
    bits, low = (11, -24) if dtype == "f16" else (8, -133)
    exponent = np.frexp(np.maximum(np.maximum(np.abs(a), np.abs(b)), 1e-300))[1]
    return np.exp2(np.maximum(exponent - bits, low) - 1.0)


# prefix lengths of several splits; up to 64 rows per KV head: the kernel whose waves split the keys
TREE_ALONE = [("bf16", 32, 8, 128, 64, 26000), ("f16", 32, 8, 128, 64, 26000), ("f16", 64, 32, 64, 40, 7000),
              ("bf16", 32, 8, 128, 16, 9000), ("f16", 8, 2, 64, 12, 9000)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,hq,hkv,d,t,plen", TREE_ALONE)
def test_the_tree_part_is_rounded_once(dtype, hq, hkv, d, t, plen):
    """The cached keys weigh nothing and every node a row sees weighs the same, so numerators are exact and a row
    is the mean of the values on its path: fp32 until it is rounded to the output type.  The bound is that
    rounding and a few fp32 ones (path length times 2^-24) of the mean of the magnitudes; f16 values are small
    enough to come out subnormal in part."""
    batch = make(dtype, hq, hkv, d, t, [plen], "iid", 35000 + t)
    seq = batch.seqs[0]
    seq.q[...] = 0.0
    seq.q[..., 0] = 4.0
    seq.k_cache[..., 0] = synth.round_to(np.float32(-60 * np.log(2) * np.sqrt(d) / 4), dtype)
    seq.k_tree[..., 0] = 0.0
    if dtype == "f16":
        seq.v_tree[...] = synth.round_to(seq.v_tree * 2.0 ** -12, dtype)
    print(f"tree alone {dtype} hq={hq} hkv={hkv} d={d} t={t} plen={plen}", flush=True)
    db = DeviceBatch(batch)
    assert ls.ls_prefix_num_splits(db.desc) > 1
    out, lse = whole_call(db)
    ro, rl = oracle_full(batch)
    assert np.abs(lse - rl).max() <= 1e-5
    seq.v_tree[...] = np.abs(seq.v_tree)
    magnitude, _ = oracle_full(batch)
    excess = (np.abs(out - ro) - half_spacing(out, ro, dtype)) / magnitude
    print(f"  beyond the output rounding: {excess.max():.2e} of the mean magnitude", flush=True)
    assert excess.max() <= 2.0 ** -20


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,hq,hkv,d,t,plen", TREE_ALONE + [("bf16", 8, 2, 128, 40, 100), ("f16", 8, 2, 64, 16, 0)])
@pytest.mark.parametrize("below", [0, 20])
def test_numerators_of_tree_keys_stay_in_fp32(dtype, hq, hkv, d, t, plen, below):
    """The cached keys weigh nothing; the nodes' scores lie within one power of two, so the arguments of the
    exponential are at most 1 and its fp32 error a few 2^-24; values of both signs cancel, so that a numerator
    rounded to 16 bits shows in the sum.  below = 20: the root outweighs the others 2^20 times and its value is zero
    (arguments up to 20, each 2^-24 of one 20 * ln 2 * 2^-24 of the numerator).  (The last two: one split.)"""
    batch = make(dtype, hq, hkv, d, t, [plen], "iid", 36000 + t)
    seq = batch.seqs[0]
    rng = np.random.default_rng(36)
    unit = np.log(2) * np.sqrt(d) / 4  # of k, per power of two of the weight
    seq.q[...] = 0.0
    seq.q[..., 0] = 4.0
    if plen:
        seq.k_cache[..., 0] = synth.round_to(np.float32(-60 * unit), dtype)
        seq.v_cache[...] = 0.0
    seq.k_tree[..., 0] = synth.round_to((-unit * rng.random(seq.k_tree.shape[:2])).astype(np.float32), dtype)
    if below:
        seq.k_tree[:, 0, 0] = synth.round_to(np.float32(below * unit), dtype)
        seq.v_tree[...] = synth.round_to(seq.v_tree * 256, dtype)
        seq.v_tree[:, 0] = 0.0
    print(f"numerators {dtype} hq={hq} hkv={hkv} d={d} t={t} plen={plen} below={below}", flush=True)
    db = DeviceBatch(batch)
    out, lse = whole_call(db)
    ro, rl = oracle_full(batch)
    assert np.abs(lse - rl).max() <= 1e-5
    seq.v_tree[...] = np.abs(seq.v_tree)
    magnitude, _ = oracle_full(batch)
    seen = magnitude > 0
    excess = ((np.abs(out - ro) - half_spacing(out, ro, dtype))[seen] / magnitude[seen]).max()
    print(f"  beyond the output rounding: {excess:.2e} of the mean magnitude", flush=True)
    assert excess <= (2.0 ** -18 if below else 2.0 ** -20)
    assert np.all(out[~seen] == 0.0)


@pytest.mark.gpu
@pytest.mark.parametrize("t,plen", [(40, 13000), (100, 6500)])
def test_bad_parents_are_cut_and_reported(t, plen):
    batch = make("bf16", 32, 8, 128, t, [plen, plen], "tree", 33000 + t)
    db = DeviceBatch(batch)
    bad = [s.parents.copy() for s in batch.seqs]
    bad[1][t // 2], bad[1][t - 1] = t - 1, -7
    cut = [p.copy() for p in bad]
    cut[1][t // 2], cut[1][t - 1] = -1, -1
    print(f"bad parents t={t} plen={plen}", flush=True)
    results = []
    for parents in (bad, cut):
        db.parents = torch.from_numpy(np.stack(parents)).cuda()
        out, lse = whole_call(db)
        at = ls.ls_workspace_error(db.desc, db.workspace) - db.workspace.data_ptr()
        results.append((out, lse, db.workspace[at:at + 8].view(torch.int32).cpu().tolist()))
    assert results[0][2] == [0, 1] and results[1][2] == [0, 0]
    assert np.array_equal(results[0][0], results[1][0]) and np.array_equal(results[0][1], results[1][1])


@pytest.mark.gpu
@pytest.mark.parametrize("lens", [[16384, 16384], [16384, 100], [16384, 0]])
def test_pieces_longer_than_a_split_are_not_dealt(lens):
    """Two sequences that fill a capacity of two splits of 8192 rows: with the tree priced in, even pieces would be longer
    than a split may be, and every sequence gets two as without dealing.  (The others are dealt.)  Against float64 on
    the device, some heads."""
    hq, d, t = 64, 64, 66
    gen = torch.Generator(device="cuda").manual_seed(16)
    new = lambda rows: torch.randn((2, hq, rows, d), generator=gen, device="cuda", dtype=torch.bfloat16)
    q, kt, vt, k, v = new(t), new(t), new(t), new(16384), new(16384)
    parents = [synth.tree_constrained(np.random.default_rng(s), t, 10, 4) for s in range(2)]
    out, lse = torch.full_like(q, float("nan")), torch.full(q.shape[:3], float("nan"), device="cuda")
    desc = ls.make_desc(q, k, v, kt, vt, out, 16384)
    assert ls.ls_prefix_num_splits(desc) == 2 and ls.ls_prefix_split_len(desc, 0) == 8192
    print(f"pieces longer than a split {lens}", flush=True)
    work = torch.full((ls.ls_workspace_bytes(desc),), 0xFF, dtype=torch.uint8, device="cuda")
    ls.ls_hybrid_tree_attn(desc, q, k, v, torch.tensor(lens, dtype=torch.int32, device="cuda"), kt, vt,
                           torch.from_numpy(np.stack(parents)).cuda(), out, lse, work)
    torch.cuda.synchronize()
    for b in range(2):
        sees = np.eye(t, dtype=bool)
        for i in range(t):
            j = i
            while j >= 0:
                sees[i, j] = True
                j = parents[b][j]
        for h in (0, 31, 63):
            keys = torch.cat([k[b, h, :lens[b]], kt[b, h]]).double()
            vals = torch.cat([v[b, h, :lens[b]], vt[b, h]]).double()
            z = (q[b, h].double() @ keys.T) / np.sqrt(d)
            z[:, lens[b]:] = z[:, lens[b]:].masked_fill(~torch.from_numpy(sees).cuda(), float("-inf"))
            ref_lse = torch.logsumexp(z, 1)
            ref = (z - ref_lse[:, None]).exp() @ vals
            gates(out[b, h].float().cpu().numpy(), lse[b, h].cpu().numpy(), ref.cpu().numpy(), ref_lse.cpu().numpy(), "bf16",
                  f"  sequence {b} head {h}", stress=True)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_neighbours_change_a_sequence_by_rounding_only(dtype):
    """Pieces are dealt by the lengths of all sequences of a call, so another neighbour moves the cuts of a sequence: each
    16-bit part, and the output, is rounded once (half an ulp of the largest value, on either side), and with the cuts
    the reference exponents of the numerators move (half an ulp, twice that where halves are cut off, again on
    either side).  The same neighbours give the same bits."""
    hq, hkv, d, t = 32, 8, 128, 40
    batch = make(dtype, hq, hkv, d, t, [5000, 6000, 6000, 6000], "peaked", 37000)
    db = DeviceBatch(batch)
    results = []
    for others in ([6000, 6000, 6000], [300, 0, 2000], [6000, 6000, 6000]):
        db.prefix_lens = torch.tensor([5000] + others, dtype=torch.int32, device="cuda")
        out, lse = db.run_full()
        torch.cuda.synchronize()
        results.append((out[0].float().cpu().numpy(), lse[0].cpu().numpy()))
    assert np.array_equal(results[0][0], results[2][0]) and np.array_equal(results[0][1], results[2][1])
    assert not np.array_equal(results[0][0], results[1][0])  # (the cuts did move)
    vmax = max(np.abs(batch.seqs[0].v_cache).max(), np.abs(batch.seqs[0].v_tree).max())
    half_ulp = 2.0 ** -11 if dtype == "f16" else 2.0 ** -8  # relative
    assert np.abs(results[0][0] - results[1][0]).max() <= 2 * (2 + (2 if dtype == "f16" else 1)) * half_ulp * vmax
    assert np.abs(results[0][1] - results[1][1]).max() <= 1e-5 * np.abs(results[0][1]).max()
