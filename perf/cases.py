"""What the extend / verify library is timed on: the calls an agent's program makes, over the decoder shapes of
`inputs.SHAPES`, through the binding's `DeviceModel`.

  extend        one session: T uncached tokens over a cached prefix of P (P = 0: the prefix itself is computed)
  verify        one session: one speculative round of k drafts over a cache of P (k = 0: plain one-token decoding)
  batch_extend  n sessions that fork one prefix of P, each with a private history, extended together
  batch_verify  the same sessions, one speculative round each in a single call

A pass cuts the caches back to where they were (what every turn and every rolled-back round does) and makes one call.
Its outputs are what the call returns and, as views of the pool's memory, the KV blocks that hold the new rows.

Weights and tokens.  A trained model mostly knows its next token; independent random matrices do not, and near-ties would
then decide which drafts are accepted.  So the LM head row of a token's successor (a seeded permutation of the vocabulary)
is a scaled copy of that token's embedding, and the embedding is large enough to survive the layers: greedy decoding
follows the permutation with a wide margin whatever the order of summation, and drafts can be right or wrong on
purpose.  All other matrices are N(0, 0.02), gains 1 + N(0, 0.02), prompts templated Zipf draws (see `inputs`).
"""
import math
import random

import numpy as np
import torch

from paper_2605_10380_amd import binding as B
from paper_2605_10380_amd import inputs as I

CHUNK = 1024                       # tokens per call while a prefix or a history is built
OUT = {"none": B.AX_OUT_NONE, "last_argmax": B.AX_OUT_LAST_ARGMAX, "last_logits": B.AX_OUT_LAST_LOGITS,
       "all_logits": B.AX_OUT_ALL_LOGITS}


def listed():
    return [
        # the fp32 exactness model: the smallest calls, launches and latency count
        {"name": "tiny_verify_k4", "kind": "verify", "shape": "tiny", "P": 512, "k": 4},
        {"name": "tiny_extend_64", "kind": "extend", "shape": "tiny", "P": 512, "T": 64, "out": "all_logits"},
        # one token at a time: what a session falls back to when the lookup table has no draft
        {"name": "1b_decode", "kind": "verify", "shape": "1b", "P": 1301, "k": 0},
        # the headline workload: the verify rounds and the turn's uncached suffix
        {"name": "1b_verify_k8", "kind": "verify", "shape": "1b", "P": 4352, "k": 8},
        {"name": "1b_extend_256", "kind": "extend", "shape": "1b", "P": 4096, "T": 256, "out": "last_argmax"},
        # a prefix that is not cached yet, in one call
        {"name": "1b_prefill_4096", "kind": "extend", "shape": "1b", "P": 0, "T": 4096, "out": "none"},
        # the longest draft, and a long tool answer, at the ~3B shape; a cache that ends inside a block
        {"name": "3b_verify_k16", "kind": "verify", "shape": "3b", "P": 6157, "k": 16},
        {"name": "3b_extend_1024", "kind": "extend", "shape": "3b", "P": 6144, "T": 1024, "out": "last_logits"},
        # the largest decoder (activations in hi + lo parts), long context
        {"name": "8b_verify_k8", "kind": "verify", "shape": "8b", "P": 8704, "k": 8},
        {"name": "8b_extend_512", "kind": "extend", "shape": "8b", "P": 8192, "T": 512, "out": "last_argmax"},
        # the plan-out agent: 16 sessions over one system prefix, ragged lengths
        {"name": "3b_batch_verify", "kind": "batch_verify", "shape": "3b", "P": 6144, "n": 16, "h_lo": 1024, "h_hi": 2048,
         "k": 8, "mix": 1},
        {"name": "3b_batch_extend", "kind": "batch_extend", "shape": "3b", "P": 6144, "n": 16, "h_lo": 1024, "h_hi": 2048,
         "t_lo": 32, "t_hi": 512, "mix": 2},
    ]


def draw(rng):
    most = [work(c) for c in listed()]
    most_bytes, most_flops = max(w["bytes"] for w in most), max(w["flops"] for w in most)

    def log_int(lo, hi):
        return min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))

    while True:
        kind = rng.choices(["verify", "extend", "batch_verify", "batch_extend"], [4, 4, 1, 1])[0]
        if kind in ("verify", "extend"):
            shape = rng.choices(["tiny", "1b", "3b", "8b"], [2, 4, 3, 1])[0]
            c = {"kind": kind, "shape": shape, "P": log_int(32, 1024 if shape == "tiny" else 8704)}
            if kind == "verify":
                c["k"] = rng.randint(0, 16)
            else:
                c["T"] = log_int(8, 256 if shape == "tiny" else 4096)
                c["out"] = rng.choice(["last_argmax", "last_logits", "none"] + (["all_logits"] if c["T"] <= 64 else []))
                if c["T"] > 1024 and rng.random() < 0.5:
                    c["P"] = 0
        else:
            h_lo, t_lo = log_int(64, 1024), log_int(8, 64)
            c = {"kind": kind, "shape": rng.choice(["1b", "3b"]), "P": log_int(256, 6144), "n": rng.randint(2, 16), "h_lo": h_lo,
                 "h_hi": 2 * h_lo, "mix": rng.randrange(1 << 20)}
            if kind == "batch_verify":
                c["k"] = rng.randint(1, 12)
            else:
                c.update(t_lo=t_lo, t_hi=8 * t_lo)
        w = work(c)
        if w["bytes"] <= most_bytes and w["flops"] <= most_flops:
            return c


def lengths(case):
    """Cached tokens and new rows of every session of the call."""
    if case["kind"] == "extend":
        return [case["P"]], [case["T"]]
    if case["kind"] == "verify":
        return [case["P"]], [1 + case["k"]]
    mix = random.Random(case["mix"])
    cached = [case["P"] + mix.randint(case["h_lo"], case["h_hi"]) for _ in range(case["n"])]
    if case["kind"] == "batch_verify":
        return cached, [1 + case["k"]] * case["n"]
    return cached, [mix.randint(case["t_lo"], case["t_hi"]) for _ in range(case["n"])]


def make_weights(sh, g):
    """Every tensor drawn on the device in its storage type, and the successor of every token."""
    dt = torch.float32 if sh.dtype == "f32" else torch.bfloat16
    out = {}
    for name, layer, dims in I.weight_names(sh):
        t = torch.empty(dims, dtype=dt, device="cuda")
        if len(dims) == 1:
            t.normal_(1.0, 0.02, generator=g)
        else:
            t.normal_(0.0, 2.0 if name == "tok_emb" else 0.02, generator=g)
        if layer is None:
            out[name] = t
        else:
            out.setdefault(name, []).append(t)
    successor = torch.randperm(sh.vocab, generator=g, device="cuda")
    out["lm_head"][successor] = out["tok_emb"] * 0.015
    return out, successor.cpu().numpy()


class State:
    def __init__(self, case, seed):
        sh = I.SHAPES[case["shape"]]
        cached, rows = lengths(case)
        g = torch.Generator(device="cuda").manual_seed(seed)
        rng = np.random.default_rng(seed)
        weights, successor = make_weights(sh, g)
        shared = case["P"]
        max_tokens = max(CHUNK, sum(rows))
        pool_tokens = shared + 64 + sum(c - shared + r + 48 for c, r in zip(cached, rows))
        self.case, self.cached, self.rows = case, cached, rows
        self.dm = dm = B.DeviceModel(sh, weights, max_pos=max(c + r for c, r in zip(cached, rows)) + 64, max_tokens=max_tokens,
                                     pool_tokens=pool_tokens, max_seqs=len(cached))
        prompt = I.templated_prompt(sh.vocab, seed, shared + 64)
        root = dm.new_kv()
        for at in range(0, shared, CHUNK):
            dm.extend(root, prompt[at:min(at + CHUNK, shared)])
        if case["kind"].startswith("batch"):
            self.kvs = [B.ax_kv_fork(root) for _ in cached]
            self.held = self.kvs + [root]
            for kv, c in zip(self.kvs, cached):
                tokens = rng.integers(0, sh.vocab, c - shared).astype(np.int32)
                for at in range(0, len(tokens), CHUNK):
                    dm.extend(kv, tokens[at:at + CHUNK])
        else:
            self.kvs = self.held = [root]
        # the call's tokens: a suffix of fresh text, or the last token and drafts of which the first few are right
        self.tokens, self.pending, self.drafts = [], [], []
        for n in rows:
            self.tokens.append(rng.integers(0, sh.vocab, n).astype(np.int32))
            chain = [int(rng.integers(0, sh.vocab))]
            for _ in range(n - 1):
                chain.append(int(successor[chain[-1]]))
            right = int(rng.integers(0, n))
            drafts = chain[1:]
            if right < len(drafts):
                drafts[right] = (drafts[right] + 1 + int(rng.integers(0, sh.vocab - 1))) % sh.vocab
            self.pending.append(chain[0])
            self.drafts.append(np.array(drafts, dtype=np.int32))
        self.new_blocks = self.views_of_new_blocks(sh)
        torch.cuda.synchronize()

    def views_of_new_blocks(self, sh):
        """The pool's memory where the call's rows will lie: [layer, K | V, KV head, blocks, elements of a block].  Blocks
        come off a stack: sequences cut back last to first get the same ones again."""
        ids = []
        for kv, n, c in zip(self.kvs, self.rows, self.cached):
            B.ax_kv_reserve_host(kv, n)
            ids += [int(b) for b in B.ax_kv_blocks(kv)[c // 16:]]
        self.cut_back()
        elements = 16 * sh.head_dim
        pool = self.dm.pool_mem.view(torch.float32 if sh.dtype == "f32" else torch.float16).view(
            sh.n_layers, 2, sh.n_kv_heads, -1, elements)
        ids.sort()
        starts = [i for i in range(len(ids)) if i == 0 or ids[i] != ids[i - 1] + 1]
        return [pool[:, :, :, ids[a]:ids[b - 1] + 1] for a, b in zip(starts, starts[1:] + [len(ids)])]

    def cut_back(self):
        for kv, c in zip(reversed(self.kvs), reversed(self.cached)):
            B.ax_kv_truncate(kv, c)

    def __del__(self):
        if getattr(self, "dm", None) is not None:
            for kv in getattr(self, "held", []):
                B.ax_kv_free(kv)
            self.dm.close()
            B.ax_pool_destroy(self.dm.pool)


def prepare(case, seed):
    return State(case, seed)


def run(state):
    kind, dm = state.case["kind"], state.dm
    state.cut_back()
    if kind == "extend":
        out = dm.extend(state.kvs[0], state.tokens[0], OUT[state.case["out"]])
    elif kind == "verify":
        out = dm.verify(state.kvs[0], state.pending[0], state.drafts[0])
    elif kind == "batch_extend":
        out = dm.extend_batch(state.kvs, state.tokens, B.AX_OUT_LAST_ARGMAX)
    else:
        accepted, after = dm.verify_batch(state.kvs, state.pending, state.drafts)
        out = np.array([accepted, after], dtype=np.int32)
    return {"result": out, "kv": state.new_blocks}


def work(case):
    """Weights once, every cached K and V once (a shared prefix once), the new rows' K and V and the outputs written."""
    sh = I.SHAPES[case["shape"]]
    cached, rows = lengths(case)
    R = sum(rows)
    verify = case["kind"].endswith("verify")
    out_rows = R if verify or case.get("out") == "all_logits" else 0 if case.get("out") == "none" else len(rows)
    kv_token = 2 * sh.n_layers * sh.n_kv_heads * sh.head_dim * sh.itemsize
    in_cache = case["P"] + sum(c - case["P"] for c in cached)
    weights = sh.n_layers * sh.layer_params + (sh.vocab * sh.d_model if out_rows else 0)
    logits_out = out_rows * sh.vocab * 4 if case.get("out") in ("last_logits", "all_logits") else out_rows * 4
    pairs = sum(t * (c + (t + 1) / 2) for c, t in zip(cached, rows))        # (row, key) pairs the causal attention scores
    return {"bytes": weights * sh.itemsize + R * sh.d_model * sh.itemsize + (in_cache + R) * kv_token + logits_out,
            "flops": 2.0 * R * sh.n_layers * sh.layer_params + 2.0 * out_rows * sh.vocab * sh.d_model
                     + 4.0 * pairs * sh.n_q_heads * sh.head_dim * sh.n_layers}


def tolerance(case):
    """fp32 models: 32-bit sums in another order.  16-bit models: fp16 activations and KV, rounded at every kernel's
    end; token ids and accepted lengths are the same (the margins are wide, see above)."""
    return {"rel": 1e-5, "max": 4e-4} if I.SHAPES[case["shape"]].dtype == "f32" else {"rel": 1e-2, "max": 0.1}
