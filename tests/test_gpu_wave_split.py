"""The whole-path kernel whose waves split the keys (few query rows per KV head, or a short cache) at the
sizes where it can go wrong: tiles of 32 keys and their remainders, rounds of eight tiles, row blocks
of 32 and 64, trees on both sides of the 64 nodes whose mask is built in registers, one split (final
output) and several (merge with the rounding remainders of the tree's split)."""
import os
import re
import subprocess
import sys

import numpy as np
import pytest
import torch

from paper_2502_17421_amd import binding as ls
from paper_2502_17421_amd import build as ls_build
from paper_2502_17421_amd import synth
from test_gpu_light_block import make
from test_gpu_paged import PagedBatch
from util import DeviceBatch, gates, oracle_full


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


# dtype, query heads, KV heads, head_dim, tree nodes, prefix lengths, inputs
CASES = [
    ("bf16", 4, 1, 128, 1, [0], "iid"),                     # one row, no cached key
    ("bf16", 8, 2, 128, 8, [1, 0, 31], "peaked"),           # 32 rows: one row tile, exactly
    ("f16", 8, 2, 128, 9, [32, 33, 257], "peaked"),         # 36 rows: two row tiles, the second nearly empty
    ("bf16", 8, 2, 64, 16, [255, 256, 1000], "tree"),       # 64 rows, rounds of eight tiles and one key beyond
    ("f16", 4, 4, 64, 32, [512, 5], "tree"),                # a KV head per query head
    ("bf16", 4, 4, 128, 33, [224, 700], "tree"),            # 33 rows and two tree tiles
    ("bf16", 16, 4, 128, 64, [300], "peaked"),              # 64 nodes: the last size masked in registers
    ("f16", 16, 4, 128, 65, [300, 11], "tree"),             # 65: the chains are walked in LDS
    ("bf16", 10, 2, 128, 130, [100], "tree"),               # five tree tiles, 650 rows
    ("bf16", 6, 2, 64, 300, [40, 0], "tree"),               # ten tree tiles: a wave has two of them
    ("bf16", 8, 2, 128, 16, [9000], "tree"),                # several splits, two row tiles
    ("f16", 8, 8, 128, 20, [6001, 17, 0], "tree"),          # several splits, sequences with fewer tiles than splits
    ("bf16", 5, 1, 64, 6, [20011], "peaked"),
    ("bf16", 8, 2, 128, 33, [1537, 3], "tree"),             # more than 64 rows, several splits: the shortest cache
    ("f16", 8, 2, 64, 70, [4256], "peaked"),                # and the longest: 133 cached tiles and 3 of the tree
    ("bf16", 32, 8, 128, 136, [2400], "tree"),              # 544 rows over 8 heads: one split of 80 tiles
]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,hq,hkv,d,t,plens,variant", CASES)
def test_whole_call_against_the_oracle(dtype, hq, hkv, d, t, plens, variant):
    if t == 1 or plens == [0]:
        batch = make(dtype, hq, hkv, d, t, plens, variant, 21000 + t)
    else:
        batch = make(dtype, hq, hkv, d, t, plens, variant, 21000 + hq + t)
    say(f"wave split {dtype} hq={hq} hkv={hkv} d={d} t={t} plens={plens} {variant}")
    db = DeviceBatch(batch, token_major=t % 2 == 0)
    out, lse = db.run_full()
    torch.cuda.synchronize()
    ro, rl = oracle_full(batch)
    say(gates(out.float().cpu().numpy(), lse.cpu().numpy(), ro, rl, dtype, "  result", stress=True))
    first = (out.clone(), lse.clone())
    db.workspace.fill_(0xFF)  # NaN bit patterns: whatever the workspace and the outputs held, the result is the same
    out.fill_(float("nan"))
    out, lse = db.run_full()
    torch.cuda.synchronize()
    assert torch.equal(out, first[0]) and torch.equal(lse, first[1])
    # the same cache in shuffled pages: bit for bit
    pb = PagedBatch(batch, 16 if t % 3 else 64, np.random.default_rng(3))
    po, pl = pb.run()
    if pb.desc.max_prefix_len == db.desc.max_prefix_len:
        assert np.array_equal(po, first[0].float().cpu().numpy()) and np.array_equal(pl, first[1].cpu().numpy())
    # cached keys only
    out, lse = db.run_cache_only()
    torch.cuda.synchronize()
    ro, rl = oracle_full(batch, use_tree=False)
    say(gates(out.float().cpu().numpy(), np.where(np.isfinite(rl), lse.cpu().numpy(), 0.0), ro,
              np.where(np.isfinite(rl), rl, 0.0), dtype, "  cached keys only", stress=True))
    assert np.array_equal(np.isfinite(rl), np.isfinite(lse.cpu().numpy()))


@pytest.mark.gpu
@pytest.mark.parametrize("t,plen", [(7, 100), (70, 100), (16, 8000)])
def test_bad_parents_are_cut_and_reported(t, plen):
    """An entry outside {-1} u [0, i) counts as -1 and sets the sequence's error word, here as everywhere."""
    batch = make("bf16", 8, 2, 128, t, [plen, plen], "tree", 22000 + t)
    good = DeviceBatch(batch)
    ref = [s.parents.copy() for s in batch.seqs]
    bad = [p.copy() for p in ref]
    bad[1][t // 2], bad[1][t - 1] = t - 1, -7
    cut = [p.copy() for p in ref]
    cut[1][t // 2], cut[1][t - 1] = -1, -1

    def run(parents):
        good.parents = torch.from_numpy(np.stack(parents)).cuda()
        out, lse = good.run_full()
        torch.cuda.synchronize()
        at = ls.ls_workspace_error(good.desc, good.workspace) - good.workspace.data_ptr()
        err = good.workspace[at:at + 8].view(torch.int32).cpu().tolist()
        return out.clone(), lse.clone(), err

    say(f"bad parents t={t} plen={plen}")
    o1, l1, e1 = run(bad)
    o2, l2, e2 = run(cut)
    assert e1 == [0, 1] and e2 == [0, 0]
    assert torch.equal(o1, o2) and torch.equal(l1, l2)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,hq,hkv,d,t,plen", [
    ("f16", 8, 2, 128, 5, 300),     # ten tiles, the tree's goes to the third wave
    ("bf16", 8, 2, 128, 8, 926),    # 29, the sixth: the halves of the workgroup change places
    ("bf16", 8, 2, 64, 8, 1500),    # 47, the eighth
    ("bf16", 8, 2, 128, 68, 512),   # three tree tiles, the first three waves
    ("f16", 8, 2, 64, 100, 150),    # four of them, the sixth to the first: they run on
    ("bf16", 4, 2, 64, 300, 700),   # ten of them, every wave
])
def test_cached_keys_are_added_up_alike_with_and_without_a_tree(dtype, hq, hkv, d, t, plen):
    """A tree whose keys have no weight (scores some 350 below the cached ones) leaves the bits of the call on the cached keys
    alone: which tiles a wave adds up, and in which order the waves are merged, does not depend on the tree."""
    batch = make(dtype, hq, hkv, d, t, [plen], "iid", 23000 + t)
    seq = batch.seqs[0]
    seq.q[..., 0] = 2.0
    seq.k_tree[..., 0] = -2000.0
    say(f"no weight {dtype} hq={hq} hkv={hkv} d={d} t={t} plen={plen}")
    db = DeviceBatch(batch)
    out, lse = db.run_cache_only()
    torch.cuda.synchronize()
    alone = out.clone(), lse.clone()
    out, lse = db.run_full()
    torch.cuda.synchronize()
    ro, rl = oracle_full(batch)
    say(gates(out.float().cpu().numpy(), lse.cpu().numpy(), ro, rl, dtype, "  result", stress=True))
    assert bool(torch.all(out == alone[0])) and bool(torch.all(lse == alone[1]))


# dtype, query heads, KV heads, head_dim, tree nodes, prefix length, runs of cached keys that score -inf, by an infinite
# component or (the last cases) by overflow.  A tile has 32 keys, tile i belongs to wave i % 8 while there is one split.
NOTHING = [
    ("bf16", 8, 2, 128, 5, 33, [(32, 33)]),                 # one row tile: a wave's first tile, one key long
    ("f16", 8, 2, 64, 5, 33, [(32, 33)]),
    ("f16", 8, 2, 128, 9, 300, [(0, 32), (288, 300)]),      # two row tiles: a whole first tile, the partial last one
    ("bf16", 8, 2, 128, 9, 700, [(64, 96), (320, 352)]),    # both tiles of wave 2
    ("bf16", 8, 2, 64, 9, 700, [(288, 320)]),               # the second tile of wave 1
    ("bf16", 8, 2, 128, 16, 40, [(0, 40)]),                 # every cached key: the tree alone is left
    ("bf16", 16, 4, 128, 40, 500, [(32, 64), (480, 500)]),  # 160 rows, one split
    ("bf16", 8, 2, 128, 8, 9000, [(0, 700), (4000, 4032), (8992, 9000)]),  # several splits, one of them whole
    ("f16", 8, 2, 128, 16, 9000, [(0, 700), (4000, 4032), (8992, 9000)]),
    ("bf16", 8, 2, 128, 33, 3000, [(0, 1600), (2000, 2032)]),              # more than 64 rows, several splits
    ("bf16", 8, 2, 128, 9, 750, [(0, 32), (320, 352), (736, 750)]),
    ("bf16", 32, 8, 128, 40, 26000, [(0, 2000), (25990, 26000)]),          # the kernel that shares tiles between waves
]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,hq,hkv,d,t,plen,runs", NOTHING)
def test_keys_that_score_minus_infinity_weigh_nothing(dtype, hq, hkv, d, t, plen, runs):
    batch = make(dtype, hq, hkv, d, t, [plen], "tree", 23000 + t + plen)
    seq = batch.seqs[0]
    seq.q[..., 0] = synth.round_to_bf16(np.abs(seq.q[..., 0]) + 2.0)
    for lo, hi in runs:
        seq.k_cache[:, lo:hi, 0] = synth.round_to_bf16(np.float32(-3e38)) if plen in (750, 26000) else -np.inf
    say(f"scores of -inf {dtype} hq={hq} hkv={hkv} d={d} t={t} plen={plen} {runs}")
    db = DeviceBatch(batch)
    out, lse = db.run_full()
    torch.cuda.synchronize()
    ro, rl = oracle_full(batch)
    say(gates(out.float().cpu().numpy(), lse.cpu().numpy(), ro, rl, dtype, "  result", stress=True))
    if runs == [(0, plen)]:
        return  # cached keys only: no key at all has weight
    out, lse = db.run_cache_only()
    torch.cuda.synchronize()
    ro, rl = oracle_full(batch, use_tree=False)
    say(gates(out.float().cpu().numpy(), lse.cpu().numpy(), ro, rl, dtype, "  cached keys only", stress=True))


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,hq,hkv,d,t,plen", [
    ("bf16", 8, 2, 128, 5, 300), ("f16", 8, 2, 64, 16, 300),        # one split
    ("bf16", 8, 2, 128, 8, 9000), ("f16", 8, 2, 128, 16, 9000),     # several splits and the merge of their parts
    ("bf16", 32, 8, 128, 40, 26000), ("f16", 32, 32, 64, 70, 7000),  # the same merge, kernel that shares tiles
])
def test_nan_reaches_the_rows_that_see_it_and_their_lse(dtype, hq, hkv, d, t, plen):
    """A NaN in a query row makes that row and its LSE NaN, a NaN in a cached key those of all rows of its KV head."""
    batch = make(dtype, hq, hkv, d, t, [plen], "tree", 24000 + t + plen)
    group = hq // hkv
    say(f"NaN {dtype} hq={hq} hkv={hkv} d={d} t={t} plen={plen}")
    for with_tree in (True, False):
        db = DeviceBatch(batch)
        run = db.run_full if with_tree else db.run_cache_only
        ro, rl = oracle_full(batch, use_tree=with_tree)
        db.q[0, hq - 1, t // 2, 7] = float("nan")
        db.k_cache[0, 0, plen // 3, 5] = float("nan")
        out, lse = run()
        torch.cuda.synchronize()
        out, lse = out.float().cpu().numpy(), lse.cpu().numpy()
        bad = np.zeros((1, hq, t), bool)
        bad[0, :group] = True
        bad[0, hq - 1, t // 2] = True
        assert np.isnan(lse[bad]).all() and np.isnan(out[bad]).all()
        say(gates(out[~bad], lse[~bad], ro[~bad], rl[~bad], dtype, "  the other rows", stress=True))


def loads_left_alone(lines):
    """Loads written in assembly return their registers to the compiler before the data is there: nothing may touch
    them between the load and the wait that follows it in the text (also in assembly)."""
    number = re.compile(r"\bv(?:\[(\d+):(\d+)\]|(\d+))")
    registers = lambda text: {r for a, b, c in number.findall(text) for r in range(int(a or c), int(b or c) + 1)}
    pending, in_asm, seen = set(), False, 0
    for ln in lines:
        if "#ASMSTART" in ln or "#ASMEND" in ln:
            in_asm = "#ASMSTART" in ln
            continue
        text = ln.split(";")[0].strip()
        if not text or text.endswith(":") or text.startswith("."):
            continue
        if in_asm and text.startswith("s_waitcnt vmcnt"):
            pending = set()
        elif in_asm and re.match(r"global_load_dword(x4)? v", text):
            dst, rest = text.split(",", 1)
            assert not registers(rest) & pending, text
            pending |= registers(dst)
            seen += 1
        else:
            if text.startswith("v_mad_u64_u32"):  # 32-bit products: the upper half of the addend reaches only that of the sum
                text = re.sub(r"v\[(\d+):\d+\]$", r"v\1", text)
            assert not registers(text) & pending, text
    assert seen > 0


def test_the_kernel_keeps_its_loads_counted(tmp_path):
    """No register spills to scratch (the kernel counts its own outstanding loads), and M0 belongs to
    the HBM -> LDS copies alone (they set it inside assembly, which cannot declare it clobbered)."""
    if not os.path.exists(ls_build.RESOURCE_REPORT) or ls_build.is_stale():
        ls_build.build_library()
    kernels = {k: v for k, v in ls_build.kernel_resources().items() if "wave_split_kernel" in k}
    assert len(kernels) >= 16
    for name, r in kernels.items():
        assert r.get("ScratchSize", 0) == 0 and r.get("VGPRs Spill", 0) == 0, (name, r)
    asm = tmp_path / "wave_split.s"
    flags = [f for f in ls_build.FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([ls_build.HIPCC, *flags, "-S", "--cuda-device-only", "-o", str(asm),
                    os.path.join(ls_build.CSRC, "ls_wave_split.hip")], check=True, stderr=subprocess.DEVNULL)
    lines = asm.read_text().splitlines()
    loads_left_alone(lines)
    copies = sum("global_load_lds_dwordx4" in ln for ln in lines)
    m0 = [ln.strip() for ln in lines if re.search(r"\bm0\b", ln.split(";")[0])]
    assert copies > 0 and len(m0) == copies
    assert all(re.fullmatch(r"s_mov_b32 m0, (s\d+|vcc_lo|vcc_hi)", ln) for ln in m0)
