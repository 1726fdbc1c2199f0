"""Performance cases: the calls that a program doing tree-speculative decoding makes of this library.

Per decoding round and layer such a program makes one verification call (hybrid tree attention over
the cached rows and the tree), a few calls of the draft model (attention over its short window, cross
attention over the target's cache), and once per round it accepts a path and moves the accepted rows
into the cache.  The cases walk these calls over the lengths a conversation passes through, over the
head layouts of the benchmark workloads (synth.WORKLOADS), over the storage types and over the two
cache layouts.

A case's "kind":
  verify   ls_hybrid_tree_attn (ls_hybrid_tree_attn_single where "single" is set)
  paged    ls_hybrid_tree_attn_paged
  cross    ls_cache_attn
  commit   ls_tree_accept_greedy, then ls_kv_commit
"""
import numpy as np
import torch

from paper_2502_17421_amd import binding as ls
from paper_2502_17421_amd import synth
from paper_2502_17421_amd.device_batch import torch_dtype

# (query heads, KV heads, head_dim) of the workloads: 8B-class GQA, 7B-class MHA, 32B-class GQA, and the
# tiny layout of the float workload
HEADS_8B, HEADS_MHA, HEADS_32B, HEADS_TINY = (32, 8, 128), (32, 32, 128), (40, 8, 128), (4, 1, 64)


def _case(name, kind, dtype, heads, batch, n_tree, tree, prefix, **options):
    """prefix: (shortest, longest) number of cached rows over the batch, both taken by some sequence."""
    case = {"name": name, "kind": kind, "dtype": dtype, "n_q_heads": heads[0], "n_kv_heads": heads[1],
            "head_dim": heads[2], "batch": batch, "n_tree": n_tree, "tree": tree,
            "prefix_lo": prefix[0], "prefix_hi": prefix[1], "capacity": prefix[1], "token_major": False,
            "single": False, "page_size": 0, "accepted": 0}
    case.update(options)
    return case


def listed():
    return [
        # The first rounds of a chat: a short prompt and a chain of five drafted tokens, f16 as served.
        _case("verify_short_chain", "verify", "f16", HEADS_8B, 1, 5, "chain", (300, 300), single=True),
        # The draft model's own attention: a sliding window of 512 rows and the 68 tokens drafted so far.
        _case("draft_window", "verify", "bf16", HEADS_8B, 1, 68, "beam", (512, 512)),
        # The float form, used to check a model's numerics: tiny heads, a random tree of 16 nodes.
        _case("verify_float", "verify", "f32", HEADS_TINY, 1, 16, "uniform", (1024, 1024)),
        # A document of 8k tokens, 64-node tree.
        _case("verify_8k", "verify", "bf16", HEADS_8B, 1, 64, "bushy", (8192, 8192)),
        # The headline: 32k tokens of context, 64-node tree.
        _case("verify_32k", "verify", "bf16", HEADS_8B, 1, 64, "bushy", (32768, 32768)),
        # No sharing of KV heads: every cached row serves one query head only.
        _case("verify_mha_16k", "verify", "bf16", HEADS_MHA, 1, 32, "bushy", (16384, 16384)),
        # The beam-search tree (widths 4, 16, 16, 16, 16) in f16 over tensors stored [B, L, H, D], at an
        # odd length of the cache.
        _case("verify_beam_f16", "verify", "f16", HEADS_8B, 1, 69, "beam", (12345, 12345), token_major=True,
              capacity=16384),
        # A static tree of 256 nodes.
        _case("verify_large_tree", "verify", "bf16", HEADS_8B, 1, 256, "bushy", (32768, 32768)),
        # Long reasoning, four sequences of unlike length in a cache of 64k rows each.
        _case("verify_long_batch", "verify", "bf16", HEADS_32B, 4, 128, "bushy", (19001, 42003), capacity=65536),
        # A serving batch: eight sequences of unlike length in pages of 16 rows.
        _case("verify_paged_batch", "paged", "bf16", HEADS_8B, 8, 24, "bushy", (501, 9003), capacity=16384,
              page_size=16),
        # One beam step of the draft model: 16 tokens attend to the target's cache.
        _case("draft_cross", "cross", "bf16", HEADS_8B, 1, 16, "chain", (32768, 32768)),
        # The end of a round: accept a path, move its rows into the cache.
        _case("accept_commit", "commit", "bf16", HEADS_32B, 4, 128, "bushy", (2000, 4000), capacity=4200, accepted=5),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    """One more case of the same ranges: short to long caches, single sequences and batches, small and
    large trees.  Anything that would cost more than verify_long_batch is drawn again."""
    limit = work(next(c for c in listed() if c["name"] == "verify_long_batch"))
    while True:
        kind = rng.choice(["verify", "verify", "verify", "window", "paged", "cross", "float", "commit"])
        heads = rng.choice([HEADS_8B, HEADS_8B, HEADS_MHA, HEADS_32B, (8, 2, 64), (16, 4, 64)])
        dtype = rng.choice(["bf16", "bf16", "f16"])
        tree = rng.choice(["bushy", "bushy", "uniform", "chain"])
        batch = rng.choice([1, 1, 1, 2, 3, 4, 8])
        options = {"token_major": rng.random() < 0.3}
        if kind == "verify":
            n_tree, hi = _log_int(rng, 4, 320), _log_int(rng, 200, 50000)
            if rng.random() < 0.25:
                batch, options["single"] = 1, True
        elif kind == "window":
            kind, n_tree, hi = "verify", _log_int(rng, 4, 90), rng.randint(64, 1100)
        elif kind == "paged":
            n_tree, hi = _log_int(rng, 4, 130), _log_int(rng, 200, 20000)
            options = {"page_size": rng.choice([16, 32, 64, 256])}
        elif kind == "cross":
            n_tree, hi = rng.randint(1, 20), _log_int(rng, 200, 50000)
        elif kind == "float":
            kind, dtype, heads = "verify", "f32", rng.choice([HEADS_TINY, HEADS_TINY, (8, 2, 128), (32, 8, 128)])
            n_tree, hi = rng.randint(1, 40), _log_int(rng, 64, 4096)
        else:
            n_tree, hi = _log_int(rng, 4, 320), _log_int(rng, 200, 4000)
            options["accepted"] = min(rng.randint(1, 8), n_tree)
        tree = "chain" if n_tree < 12 else tree
        if tree == "chain" and n_tree > 60:
            tree = "bushy"
        lo = hi if batch == 1 else max(1, int(hi * rng.uniform(0.05, 1.0)))
        capacity = hi + rng.choice([0, 0, n_tree, 64]) if kind != "commit" else hi + n_tree
        if kind != "commit" and rng.random() < 0.25:
            capacity = int(hi * rng.uniform(1.0, 2.0))
        case = _case("", kind, dtype, heads, batch, n_tree, tree, (lo, hi), capacity=capacity, **options)
        del case["name"]
        cost = work(case)
        rows = batch * capacity * heads[1] * heads[2]
        if cost["bytes"] <= limit["bytes"] and cost["flops"] <= limit["flops"] and rows <= 4 * 65536 * 8 * 128:
            return case


def _lengths(case):
    """Cached rows of the sequences, spread over [prefix_lo, prefix_hi] with both ends taken."""
    n, lo, hi = case["batch"], case["prefix_lo"], case["prefix_hi"]
    return [hi] if n == 1 else [lo + (hi - lo) * i // (n - 1) for i in range(n)]


def _tree(rng, kind, n):
    if kind == "chain":
        return synth.tree_chain(n)
    if kind == "uniform":
        return synth.tree_uniform(rng, n)
    if kind == "beam":  # the widths of the beam search, cut to n nodes in all
        return synth.tree_beam(rng)[:n]
    return synth.tree_constrained(rng, n, 12, 4)


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dtype = torch_dtype(case["dtype"])
    b, hq, hkv = case["batch"], case["n_q_heads"], case["n_kv_heads"]
    t, d, cap = case["n_tree"], case["head_dim"], case["capacity"]

    def tensor(heads, rows):
        """[B, H, L, D] view of normal values, stored [B, H, L, D] or [B, L, H, D]."""
        shape = (b, rows, heads, d) if case["token_major"] else (b, heads, rows, d)
        x = torch.randn(shape, generator=gen, device="cuda", dtype=dtype)
        return x.transpose(1, 2) if case["token_major"] else x

    lengths = [_lengths(case)[i] for i in rng.permutation(b)]
    trees = [_tree(rng, case["tree"], t) for _ in range(b)]
    st = {"case": case, "q": tensor(hq, t), "k_tree": tensor(hkv, t), "v_tree": tensor(hkv, t),
          "parents": torch.from_numpy(np.stack(trees)).cuda(),
          "prefix_lens": torch.tensor(lengths, dtype=torch.int32, device="cuda"), "prefix_len": lengths[0]}
    st["out"] = torch.zeros_like(st["q"])
    st["lse"] = torch.zeros((b, hq, t), dtype=torch.float32, device="cuda")

    if case["kind"] == "paged":
        # a pool of pages handed out in random order, as after some time of serving
        size = case["page_size"]
        per_seq = (cap + size - 1) // size
        pool = sum((n + size - 1) // size for n in lengths) + 8
        st["k"] = torch.randn((pool, hkv, size, d), generator=gen, device="cuda", dtype=dtype)
        st["v"] = torch.randn((pool, hkv, size, d), generator=gen, device="cuda", dtype=dtype)
        table, order, used = np.zeros((b, per_seq), dtype=np.int32), rng.permutation(pool), 0
        for i, n in enumerate(lengths):
            pages = (n + size - 1) // size
            table[i, :pages] = order[used:used + pages]
            used += pages
        st["table"] = torch.from_numpy(table).cuda()
    else:
        st["k"], st["v"] = tensor(hkv, cap), tensor(hkv, cap)
    st["desc"] = ls.make_desc(st["q"], st["k"], st["v"], st["k_tree"], st["v_tree"], st["out"], cap)

    if case["kind"] == "commit":
        # a draft that agrees with the target along one path of the wanted length (or down to a leaf)
        draft = rng.integers(0, 32000, size=(b, t)).astype(np.int32)
        target = rng.integers(0, 32000, size=(b, t)).astype(np.int32)
        for s, parents in enumerate(trees):
            depth = synth.tree_depths(parents)
            node = int(rng.choice(np.nonzero(depth == min(case["accepted"] - 1, depth.max()))[0]))
            while parents[node] >= 0:
                draft[s, node] = target[s, parents[node]]
                node = int(parents[node])
        st["draft"], st["target"] = torch.from_numpy(draft).cuda(), torch.from_numpy(target).cuda()
        st["path"] = torch.zeros((b, t), dtype=torch.int32, device="cuda")
        for key in ("n_accepted", "next_token", "new_lens", "err_accept", "err_commit"):
            st[key] = torch.zeros((b,), dtype=torch.int32, device="cuda")
    else:
        st["workspace"] = torch.empty(ls.ls_workspace_bytes(st["desc"]), dtype=torch.uint8, device="cuda")
    return st


def run(st):
    case = st["case"]
    if case["kind"] == "commit":
        ls.ls_tree_accept_greedy(st["parents"], st["draft"], st["target"], st["path"], st["n_accepted"],
                                 st["next_token"], st["err_accept"])
        ls.ls_kv_commit(st["desc"], st["k_tree"], st["v_tree"], st["path"], st["n_accepted"], st["prefix_lens"],
                        st["k"], st["v"], st["new_lens"], st["err_commit"])
        return [st[key] for key in ("path", "n_accepted", "next_token", "new_lens", "err_accept", "err_commit",
                                    "k", "v")]
    if case["kind"] == "cross":
        ls.ls_cache_attn(st["desc"], st["q"], st["k"], st["v"], st["prefix_lens"], st["out"], st["lse"],
                         st["workspace"])
    elif case["kind"] == "paged":
        ls.ls_hybrid_tree_attn_paged(st["desc"], st["q"], st["k"], st["v"], st["table"], case["page_size"],
                                     st["prefix_lens"], st["k_tree"], st["v_tree"], st["parents"], st["out"],
                                     st["lse"], st["workspace"])
    elif case["single"]:
        ls.ls_hybrid_tree_attn_single(st["desc"], st["q"], st["k"], st["v"], st["prefix_len"], st["k_tree"],
                                      st["v_tree"], st["parents"], st["out"], st["lse"], st["workspace"])
    else:
        ls.ls_hybrid_tree_attn(st["desc"], st["q"], st["k"], st["v"], st["prefix_lens"], st["k_tree"], st["v_tree"],
                               st["parents"], st["out"], st["lse"], st["workspace"])
    return [st["out"], st["lse"]]


def work(case):
    b, hq, hkv, t, d = (case[key] for key in ("batch", "n_q_heads", "n_kv_heads", "n_tree", "head_dim"))
    size = 4 if case["dtype"] == "f32" else 2
    if case["kind"] == "commit":
        # parents and both token arrays in, the path out, the accepted K and V rows read and written
        return {"bytes": 4 * 4 * b * t + 4 * b * case["accepted"] * hkv * d * size, "flops": 0}
    cached = sum(_lengths(case))
    # cached K and V rows, q and out, the LSEs
    n_bytes = 2 * hkv * cached * d * size + 2 * b * hq * t * d * size + 4 * b * hq * t
    flops = 4 * hq * t * cached * d
    if case["kind"] == "paged":
        n_bytes += 4 * (cached // case["page_size"])
    if case["kind"] != "cross":
        # tree K and V rows and the parents; every node sees itself and, on average, its parent at least
        n_bytes += 2 * b * hkv * t * d * size + 4 * b * t
        flops += 4 * b * hq * (2 * t - 1) * d
    return {"bytes": n_bytes, "flops": flops}


def tolerance(case):
    """Four times the error measured against the same attention in float64 over these cases and two dozen
    drawn ones (2-norm; largest single difference over the result's root mean square): bf16 2.9e-3 and
    2.4e-2, f16 5.1e-4 and 2.7e-3, f32 4.4e-7 and 2.6e-6.  The commit moves bytes."""
    if case["kind"] == "commit":
        return "exact"
    return {"bf16": {"rel": 1.2e-2, "max": 9.5e-2}, "f16": {"rel": 2e-3, "max": 1.1e-2},
            "f32": {"rel": 1.8e-6, "max": 1.05e-5}}[case["dtype"]]
