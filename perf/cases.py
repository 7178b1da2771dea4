"""Performance cases of the shallow-fusion decode path.

Each case is one call pattern of a streaming Transducer decoder through the
package's public entry points: single decode steps, greedy and beam frame
loops, the joint projection, and the projected frame loop with end-of-stream
scores.  Language models, phrase lists and logits are synthetic and seeded;
models and phrase trees are loaded once per process, as a server does, and the
logits, hidden states and hypothesis states come from the case's seed.

Logits come in two kinds.  "noise" is N(0, 2) with +2 on blank (and +8 on one
token of a tenth of the rows where ``peaked`` is set), the distribution of the
package's benchmark.  "speech" is N(0, 1) with +10 on the frame's token, blank
or emitted in equal shares, the emitted tokens following the LM's corpus, as a
trained acoustic model produces.
"""

from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_2609_14991_amd as F

BLANK = 0
LAM, BETA = 0.5, 0.5  # fusion weights of the paper's set-up
SECOND = 0.3          # weight of a second (keyword) LM


def listed():
    return [
        # the smallest call: one hypothesis, one frame, as an on-device recogniser steps
        dict(name="step_single", kind="step", H=1, V=128, N=3, n_lm=1, phrases=10, k=1, compete=False, fused=False),
        # one frame of a 64-stream x 4-slot beam kept by the caller's own beam search
        dict(name="step_frame", kind="step", H=256, V=4096, N=5, n_lm=1, phrases=10000, k=4, compete=True,
             fused=False),
        # rescoring of an odd-sized vocabulary with the whole fused row handed back
        dict(name="step_ragged_rows", kind="step", H=777, V=1001, N=4, n_lm=1, phrases=1000, k=8, compete=True,
             fused=True),
        # one live stream fed in 1040 ms look-ahead chunks of 13 frames
        dict(name="stream_chunks", kind="run", S=1, B=1, T=260, chunk=13, V=1024, N=4, n_lm=1, phrases=100, k=1,
             compete=False, logits="speech", peaked=False, recombine=False, end=False),
        # 64 streams decoded greedily, utterance by utterance
        dict(name="greedy_batch", kind="run", S=64, B=1, T=500, chunk=0, V=1024, N=4, n_lm=1, phrases=1000, k=1,
             compete=False, logits="noise", peaked=True, recombine=False, end=False),
        # a test set of 285 short utterances with a user's 300-term list
        dict(name="greedy_keyword", kind="run", S=285, B=1, T=63, chunk=0, V=1024, N=4, n_lm=1, phrases=300, k=1,
             compete=False, logits="speech", peaked=False, recombine=False, end=False),
        # the widest sub-word vocabulary, blank competing with the fused keys
        dict(name="greedy_wide", kind="run", S=32, B=1, T=120, chunk=0, V=8190, N=3, n_lm=1, phrases=1000, k=1,
             compete=True, logits="speech", peaked=False, recombine=False, end=False),
        # the benchmark's beam: 64 streams x 4 slots, 4096 tokens, 5-gram, 10,000 phrases
        dict(name="beam", kind="run", S=64, B=4, T=300, chunk=0, V=4096, N=5, n_lm=1, phrases=10000, k=4,
             compete=True, logits="noise", peaked=False, recombine=False, end=False),
        # a 6-gram beam over a small vocabulary
        dict(name="beam_6gram", kind="run", S=32, B=4, T=250, chunk=0, V=1024, N=6, n_lm=1, phrases=1000, k=4,
             compete=True, logits="speech", peaked=False, recombine=False, end=False),
        # a general and a keyword LM, recombining beam, </s> terms at the end of the streams
        dict(name="beam_two_lms", kind="run", S=23, B=8, T=60, chunk=0, V=2500, N=4, n_lm=2, phrases=300, k=8,
             compete=True, logits="speech", peaked=False, recombine=True, end=True),
        # the joint projection of every frame of a batch at once (76,800 hypothesis-frames)
        dict(name="project_batch", kind="project", M=76800, V=4096, K=640, bias=True),
        # joint projection and beam together, one 13-frame encoder chunk at a time
        dict(name="projected_chunks", kind="projected", S=64, B=4, T=39, chunk=13, V=4096, N=5, n_lm=1,
             phrases=10000, k=4, K=640, compete=True, recombine=False),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _max_order(V):
    # packed n-gram keys of the corpus counts stay below 2^63; wide vocabularies
    # keep to the orders whose tables a test box builds in seconds
    return 6 if V <= 1024 else 5 if V <= 2048 else 4 if V <= 4096 else 3


def draw(rng):
    kind = rng.choice(["step", "greedy", "greedy", "beam", "beam", "project", "projected"])
    if kind == "project":
        K = 8 * _log_int(rng, 16, 128)
        V = _log_int(rng, 128, 8190)
        most = 76800 * 4096 * 640 // (V * K)
        return dict(kind="project", M=_log_int(rng, 16, max(16, min(76800, most))), V=V, K=K, bias=rng.random() < 0.7)
    V = _log_int(rng, 128, 8190)
    n_lm = 2 if (V <= 2500 and rng.random() < 0.3) else 1
    c = dict(kind="run", V=V, N=rng.randint(3, _max_order(V)), n_lm=n_lm, phrases=_log_int(rng, 10, 10000))
    if kind == "step":
        compete = rng.random() < 0.6
        c.update(kind="step", H=_log_int(rng, 1, 4096), k=rng.choice([1, 2, 4, 8]) if compete else 1, compete=compete,
                 fused=rng.random() < 0.4)
        return c
    speech = "speech" if rng.random() < 0.6 else "noise"
    cap = 76800 * 4096  # scores of the largest listed run
    if kind == "greedy":
        S = _log_int(rng, 1, 300)
        T = max(13, min(_log_int(rng, 26, 500), cap // (4 * S * V)))
        c.update(S=S, B=1, T=T, chunk=13 if rng.random() < 0.4 else 0, k=1, compete=rng.random() < 0.3,
                 logits=speech, peaked=rng.random() < 0.5, recombine=False, end=rng.random() < 0.3)
        return c
    B, k = rng.choice([2, 3, 4, 8, 16]), rng.choice([2, 4, 8])
    S = max(1, min(_log_int(rng, 1, 64), 256 // B))
    if kind == "beam":
        recombine = rng.random() < 0.3
        # a frame takes longer the wider the vocabulary and the more candidates merge
        most = 1250 // (8 + V // 1024 + (B * k // 2 if recombine else B * k // 16))
        c.update(S=S, B=B, T=_log_int(rng, 13, max(14, most)), chunk=13 if rng.random() < 0.3 else 0, k=k,
                 compete=True, logits=speech, peaked=False, recombine=recombine, end=rng.random() < 0.3)
        return c
    chunk = rng.choice([1, 4, 13, 26])
    c.update(kind="projected", S=S, B=B, T=_log_int(rng, 13, 39), chunk=chunk, k=k, K=8 * _log_int(rng, 16, 128),
             compete=True, recombine=rng.random() < 0.3)
    return c


# ---------------------------------------------------------------------------
# models and phrase lists (made once per process)
# ---------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) & 0x7FFFFFFFFFFFFFFF)


def _zipf(g, shape, V, s=1.05):
    """Truncated-Zipf token ids 1..V-1 (blank 0 excluded)."""
    p = torch.arange(1, V, device="cuda", dtype=torch.float64) ** -s
    cdf = torch.cumsum(p / p.sum(), 0)
    r = torch.rand(shape, generator=g, device="cuda", dtype=torch.float64)
    return torch.searchsorted(cdf, r).clamp_(max=V - 2) + 1


class Model:
    """A backoff n-gram model of a Zipf corpus (absolute discounting, interpolated),
    its raw tables on the GPU, and the library's handle for it."""

    def __init__(self, V, N, seed, n_tok):
        self.V, self.N, self.base = V, N, V + 2
        base, D = self.base, 0.75
        g = _gen(seed)
        n_sent = max(50, n_tok // 18)
        lens = torch.randint(5, 31, (n_sent,), generator=g, device="cuda")
        col = torch.arange(32, device="cuda")
        sent = torch.full((n_sent, 32), -1, device="cuda", dtype=torch.int64)
        sent[:, 1:31] = _zipf(g, (n_sent, 30), V)
        sent[:, 0] = V  # <s>
        sent = torch.where(col[None] <= lens[:, None], sent, -1)
        sent.scatter_(1, lens[:, None] + 1, V + 1)  # </s>
        self.text = sent[(sent >= 0) & (sent < V)]  # the corpus' tokens in order
        self.keys, self.p, self.backoff = [None] * (N + 1), [None] * (N + 1), [None] * (N + 1)
        self.first, self.count = [None] * (N + 1), [None] * (N + 1)  # successors in the next order
        win = sent.clone()
        for k in range(1, N + 1):
            if k > 1:
                nxt = sent[:, k - 1:]
                win = torch.where(nxt >= 0, win[:, :nxt.shape[1]] * base + nxt, -1)
            u, c = torch.unique(win[win >= 0], return_counts=True)
            c = c.double()
            if k == 1:
                cnt = torch.zeros(base, device="cuda", dtype=torch.float64)
                cnt[u] = c
                ids = torch.tensor([t for t in range(V) if t != BLANK] + [V, V + 1], device="cuda")
                cnt[V] = 0.0  # <s> is a context only
                p = (cnt[ids] + 0.5) / (cnt[ids].sum() + 0.5 * (V + 1))
                p[ids == V] = 1e-43
                self.keys[1], self.p[1] = ids, p
            else:
                low = self.keys[k - 1]
                ci = torch.searchsorted(low, u // base)
                suf = torch.searchsorted(low, u % base ** (k - 1))
                tot = torch.zeros(low.numel(), device="cuda", dtype=torch.float64).scatter_add_(0, ci, c)
                types = torch.bincount(ci, minlength=low.numel())
                gamma = torch.where(types > 0, D * types / tot, torch.ones_like(tot))
                self.keys[k] = u
                self.p[k] = (c - D) / tot[ci] + gamma[ci] * self.p[k - 1][suf]
                self.backoff[k - 1] = gamma.log().float()
                self.count[k - 1] = types
                self.first[k - 1] = torch.cumsum(types, 0) - types
        self.p = [None] + [q.log().float() for q in self.p[1:]]
        toks = []
        for k in range(1, N + 1):
            d = [(self.keys[k] // base ** (k - 1 - j)) % base for j in range(k)]
            toks.append(torch.stack(d, 1).int().cpu().numpy())
        self.handle = F.ngram_load(N, V, BLANK, toks, [q.cpu().numpy() for q in self.p[1:]],
                                   [None if b is None else b.cpu().numpy() for b in self.backoff[1:]])
        self.off = [0, 0, V + 2]  # first state id of each order
        for k in range(2, N):
            self.off.append(self.off[k] + self.keys[k].numel())

    def history(self, H):
        """The start history <s> of H hypotheses: the last N-1 tokens, -1 for none."""
        h = torch.full((H, self.N - 1), -1, device="cuda", dtype=torch.int64)
        h[:, -1] = self.V
        return h

    def states(self, H, g):
        """H states a decode visits: contexts of every length drawn from the corpus text."""
        m = torch.randint(1, self.N, (H,), generator=g, device="cuda")
        at = torch.randint(0, self.text.numel() - self.N, (H,), generator=g, device="cuda")
        h = self.text[at[:, None] + torch.arange(self.N - 1, device="cuda")]
        h = torch.where(torch.arange(self.N - 1, device="cuda")[None] >= (self.N - 1 - m)[:, None], h, -1)
        ids = h[:, -1].clone()
        for k in range(2, self.N):
            key = self.context(h, k)
            i = torch.searchsorted(self.keys[k], key).clamp_(max=self.keys[k].numel() - 1)
            ids = torch.where(self.keys[k][i] == key, self.off[k] + i, ids)
        return h, ids.int()

    def context(self, h, k):
        """Packed keys of the last k tokens of each history, -1 where it is shorter."""
        key = torch.zeros(h.shape[0], device="cuda", dtype=torch.int64)
        for j in range(k):
            key = key * self.base + h[:, h.shape[1] - k + j]
        return torch.where((h[:, h.shape[1] - k:] >= 0).all(1), key, -1)

    def rows(self, h):
        """log p(y | history) of every id y < V + 2 by the backoff recursion, in float64."""
        row = torch.zeros(h.shape[0], self.base, device="cuda", dtype=torch.float64)
        row[:, self.keys[1]] = self.p[1].double()
        for k in range(1, self.N):
            key = self.context(h, k)
            i = torch.searchsorted(self.keys[k], key).clamp_(max=self.keys[k].numel() - 1)
            found = self.keys[k][i] == key
            row += torch.where(found, self.backoff[k][i].double(), 0.0)[:, None]
            who, at = _spread(self.first[k][i], torch.where(found, self.count[k][i], 0))
            row[who, self.keys[k + 1][at] % self.base] = self.p[k + 1][at].double()
        return row


def _spread(first, count):
    """Row index and position of every element of the ragged ranges [first, first + count)."""
    who = torch.repeat_interleave(torch.arange(count.numel(), device="cuda"), count)
    ends = torch.cumsum(count, 0)
    at = torch.arange(who.numel(), device="cuda") - (ends - count)[who] + first[who]
    return who, at


class Phrases:
    """A user word list: half in-corpus terms, half rare ones; its automaton and the library's handle."""

    def __init__(self, V, n, text, seed):
        self.base = base = V + 2
        rng = np.random.default_rng(seed)
        text = text[:200000].cpu().numpy()
        out = []
        for i in range(n):
            L = int(rng.integers(2, 9))
            if i % 2 == 0:
                a = int(rng.integers(0, text.size - L))
                out.append(text[a:a + L])
            else:
                out.append(rng.integers(V // 2, V, size=L))
        lens = np.array([len(p) for p in out])
        offs = np.concatenate([[0], np.cumsum(lens)])
        self.handle = F.boost_build(V, BLANK, np.concatenate(out), offs)
        # nodes numbered by (depth, tokens): the ids of the package's contract
        tok = np.full((n, 8), -1, dtype=np.int64)
        for i, p in enumerate(out):
            tok[i, :len(p)] = p
        at = np.zeros(n, dtype=np.int64)
        depth, bonus, edges, child = [0], [0.0], [], []
        for d in range(8):
            live = lens > d
            e, inv = np.unique(at[live] * base + tok[live, d], return_inverse=True)
            at[live] = len(depth) + inv.reshape(-1)
            b = np.zeros(e.size)
            b[np.unique(at[lens == d + 1]) - len(depth)] = d + 1.0
            edges.append(e)
            child.append(len(depth) + np.arange(e.size))
            depth += [d + 1] * e.size
            bonus += b.tolist()
        edge, child = np.concatenate(edges), np.concatenate(child)
        depth, bonus = np.array(depth), np.array(bonus)
        parent, word = edge // base, edge % base  # edge i leads to node child[i] = i + 1
        fail, out_sum = np.zeros(depth.size, dtype=np.int64), np.zeros(depth.size)
        for d in range(1, 9):
            ids = np.nonzero(depth == d)[0]
            f = fail[parent[ids - 1]]
            todo = np.ones(ids.size, dtype=bool) if d > 1 else np.zeros(ids.size, dtype=bool)
            while todo.any():
                key = f * base + word[ids - 1]
                i = np.minimum(np.searchsorted(edge, key), edge.size - 1)
                hit = todo & (edge[i] == key)
                fail[ids[hit]] = child[i[hit]]
                todo &= ~hit & (f != 0)
                f = fail[f]
            out_sum[ids] = bonus[ids] + out_sum[fail[ids]]
        phi = np.where(bonus > 0, 0.0, depth)
        dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
        self.n_nodes, self.depth = depth.size, 8
        self.edge, self.fail, self.phi, self.E = dev(edge), dev(fail), dev(phi), dev(phi + out_sum)
        n_child = np.bincount(parent, minlength=depth.size)
        self.count, self.first = dev(n_child), dev(np.cumsum(n_child) - n_child)

    def rows(self, q):
        """The phrase state after every token (float64 boost, next node), from states q."""
        nxt = torch.zeros(q.numel(), self.base, device="cuda", dtype=torch.int64)
        chain = [q]
        for _ in range(self.depth):
            chain.append(self.fail[chain[-1]])
        root = torch.zeros_like(q)
        for i, node in enumerate([root] + chain[::-1]):
            cnt = self.count[node] if i == 0 else torch.where(node > 0, self.count[node], 0)
            who, at = _spread(self.first[node], cnt)
            nxt[who, self.edge[at] % self.base] = at + 1
        return self.E[nxt] - self.phi[q][:, None], nxt


@functools.lru_cache(maxsize=None)
def _model(V, N, which=0):
    # about a thousand tokens a word; a keyword LM is estimated from a tenth of that
    return Model(V, N, 2609 + 7 * which, min(4_000_000, 1000 * V) // (10 if which else 1))


@functools.lru_cache(maxsize=None)
def _phrases(V, N, n):
    return Phrases(V, n, _model(V, N).text, 14991)


def _models(case):
    ms = [_model(case["V"], case["N"])]
    if case["n_lm"] == 2:
        ms.append(_model(case["V"], min(4, case["N"]), 1))
    return ms, [LAM, SECOND][:case["n_lm"]]


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _logits(g, kind, peaked, T, S, B, V, text):
    """[T, S * B, V] float32 joint outputs."""
    H = S * B
    x = torch.randn((T, H, V), generator=g, device="cuda")
    if kind == "noise":
        x.mul_(2.0)
        x[:, :, BLANK] += 2.0
        if peaked:
            hit = torch.rand((T, H, 1), generator=g, device="cuda") < 0.1
            tok = torch.randint(1, V, (T, H, 1), generator=g, device="cuda")
            x.scatter_add_(2, tok, hit.float() * 8.0)
        return x
    # the slots of a stream hear the same token
    emit = torch.rand((T, S), generator=g, device="cuda") < 0.5
    at = torch.cumsum(emit, 0) + torch.randint(0, text.numel() - T - 1, (S,), generator=g, device="cuda")
    tok = torch.where(emit, text[at], BLANK).repeat_interleave(B, 1)
    return x.scatter_add_(2, tok[:, :, None], torch.full((T, H, 1), 10.0, device="cuda"))


def _projection(g, M, V, K, bias=True):
    A = torch.randn((M, K), generator=g, device="cuda").bfloat16()
    W = (torch.randn((V, K), generator=g, device="cuda") * (2.0 / math.sqrt(K))).bfloat16()
    b = torch.randn(V, generator=g, device="cuda") * 0.1
    b[BLANK] += 2.0
    return A, W, b if bias else None


def _ints(*shape):
    return torch.empty(shape, dtype=torch.int32, device="cuda")


def prepare(case, seed):
    g = _gen(seed * 1000003 + 17)
    st = dict(case=case)
    kind, V = case["kind"], case["V"]
    if kind == "project":
        st["A"], st["W"], st["bias"] = _projection(g, case["M"], V, case["K"], case["bias"])
        st["out"] = torch.empty((case["M"], V), device="cuda")
        return st
    st["models"], st["alphas"] = _models(case)
    st["phr"] = _phrases(V, case["N"], case["phrases"])
    n, k = case["n_lm"], case["k"]
    if kind == "step":
        H = case["H"]
        st["x"] = _logits(g, "noise", True, 1, H, 1, V, None)[0]
        st["hist"], ids = zip(*[m.states(H, g) for m in st["models"]])
        st["lm"] = torch.stack(ids).contiguous()
        # most hypotheses are outside any phrase
        q = torch.randint(0, st["phr"].n_nodes, (H,), generator=g, device="cuda")
        st["boost"] = torch.where(torch.rand(H, generator=g, device="cuda") < 0.7, 0, q).int()
        st.update(tokens=_ints(H, k), scores=torch.empty((H, k), device="cuda"), next_lm=_ints(n, H, k),
                  next_boost=_ints(H, k), fused=torch.empty((H, V), device="cuda") if case["fused"] else None)
        return st
    S, B, T = case["S"], case["B"], case["T"]
    H = S * B
    if kind == "run":
        st["x"] = _logits(g, case["logits"], case["peaked"], T, S, B, V, st["models"][0].text)
    else:
        st["A"], st["W"], st["bias"] = _projection(g, T * H, V, case["K"])
        st["x"] = torch.empty((min(case["chunk"], T), H, V), device="cuda")
    st["lm0"] = torch.full((n, H), V, dtype=torch.int32, device="cuda")
    st["boost0"] = torch.zeros(H, dtype=torch.int32, device="cuda")
    st["lm"], st["boost"], st["tokens"], st["parents"] = _ints(n, H), _ints(H), _ints(T, H), None
    if B > 1:
        st["parents"] = _ints(T, H)
        s0 = torch.full((S, B), -math.inf, dtype=torch.float64, device="cuda")
        s0[:, 0] = 0.0
        st["score0"], st["score"] = s0.reshape(-1), torch.empty(H, dtype=torch.float64, device="cuda")
    if case["recombine"]:
        st["merge"] = torch.zeros(H, dtype=torch.int64, device="cuda")
    if kind == "run" and case["end"]:
        st["end"] = torch.empty(H, dtype=torch.float64, device="cuda")
    return st


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(st):
    case = st["case"]
    kind, V = case["kind"], case["V"]
    if kind == "project":
        F.joint_project(st["A"], st["W"], st["bias"], case["M"], V, case["K"], st["out"])
        return st["out"]
    mode = F.FUSION_BLANK_COMPETE if case["compete"] else F.FUSION_BLANK_AM
    lms, trie, k = [m.handle for m in st["models"]], st["phr"].handle, case["k"]
    if kind == "step":
        if case["n_lm"] == 1:
            F.fusion_step(lms[0], trie, st["x"], st["lm"], st["boost"], case["H"], V, LAM, BETA, BLANK, k, mode,
                          st["fused"], st["tokens"], st["scores"], st["next_lm"], st["next_boost"])
        else:
            F.fusion_step_lms(lms, st["alphas"], trie, st["x"], st["lm"], st["boost"], case["H"], V, BETA, BLANK, k,
                              mode, st["fused"], st["tokens"], st["scores"], st["next_lm"], st["next_boost"])
        out = dict(tokens=st["tokens"], scores=st["scores"], next_lm=st["next_lm"], next_boost=st["next_boost"])
        if case["fused"]:
            out["fused"] = st["fused"]
        return out
    # the streams start: <s>, no phrase, one live hypothesis each
    S, B, T = case["S"], case["B"], case["T"]
    score, hist, parents, flags = st.get("score"), st.get("merge"), st["parents"], 0
    st["lm"].copy_(st["lm0"])
    st["boost"].copy_(st["boost0"])
    if B > 1:
        score.copy_(st["score0"])
    if case["recombine"]:
        hist.zero_()
        flags = F.FUSION_RUN_RECOMBINE
    out = dict(tokens=st["tokens"], lm=st["lm"], boost=st["boost"])
    if B > 1:
        out.update(parents=parents, score=score)
    if kind == "projected":
        F.fusion_run_projected(lms, st["alphas"], trie, st["A"], st["W"], st["bias"], case["K"], st["x"],
                               case["chunk"], T, S, B, V, k, BETA, BLANK, mode, st["lm"], st["boost"], score,
                               st["tokens"], parents, flags, hist)
        out["logits"] = st["x"]
        return out
    chunk = case["chunk"] or T
    for t in range(0, T, chunk):
        n = min(chunk, T - t)
        F.fusion_run_lms(lms, st["alphas"], trie, st["x"][t:t + n], n, S, B, V, k, BETA, BLANK, mode, st["lm"],
                         st["boost"], score, st["tokens"][t:t + n], None if parents is None else parents[t:t + n],
                         flags=flags, hist=hist)
    if case["end"]:
        # added to the beam's scores, and reported by itself
        F.fusion_end_scores(lms, st["alphas"], st["lm"], S * B, score, st["end"])
        out["end"] = st["end"]
    return out


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    kind, V = case["kind"], case["V"]
    if kind == "project":
        M, K = case["M"], case["K"]
        return dict(bytes=2 * (M + V) * K + 4 * M * V + 4 * V * case["bias"], flops=2 * M * V * K)
    steps = case["H"] if kind == "step" else case["T"] * case["S"] * case["B"]
    # the logits, one LM row a hypothesis-step (never more than the model's rows), the phrase tree's root row
    lm = case["n_lm"] * min(steps, V + 2) * 4 * V
    flops = (3 * case["n_lm"] + 8) * steps * V
    if kind == "step":
        out = steps * case["k"] * 4 * (3 + case["n_lm"]) + (4 * V * steps if case["fused"] else 0)
    else:
        out = steps * 4 * (2 if case["B"] > 1 else 1)
    b = dict(bytes=4 * steps * V + lm + 4 * V + out, flops=flops)
    if kind == "projected":
        # the hidden states and the weight instead of the logits; the last chunk's logits leave the call
        K, H = case["K"], case["S"] * case["B"]
        b["bytes"] += 2 * (steps + V) * K + 4 * V * H * min(case["chunk"], case["T"]) - 4 * steps * V
        b["flops"] += 2 * steps * V * K
    return b


def tolerance(case):
    # about four times what the float64 reference, and the same decode with its
    # log-sum-exp or projection rounded otherwise, differ by
    if case["kind"] == "project":
        # fp32 sums of exact bf16 products in any order: 1.5e-7
        return {"rel": 6e-7}
    if case["kind"] == "step":
        # fp32 keys are fixed operation by operation, only the log-sum-exp's order is free: 6e-8
        return {"rel": 2.5e-7, "differ": 0.0}
    if case["kind"] == "run" and case["B"] == 1:
        # greedy decisions compare keys alone
        return {"rel": 2e-7, "differ": 0.0}
    # totals carry the log-sum-exp's (and the projection's) rounding, and a near tie that falls the
    # other way changes a stream's tokens until its paths meet again: 1.5e-7 and 1e-4 of the tokens
    return {"rel": 6e-7, "differ": 5e-4}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------
def _keys(st, x, hist, q):
    """float64 keys and fused scores [H, V] and the phrase state after every token."""
    V = x.shape[1]
    x = x.double()
    key = x.clone()
    for m, a, h in zip(st["models"], st["alphas"], hist):
        key += float(np.float32(a)) * m.rows(h)[:, :V]
    boost, nxt = st["phr"].rows(q)
    key += BETA * boost[:, :V]
    key[:, BLANK] = x[:, BLANK]
    return key, key - torch.logsumexp(x, 1)[:, None], nxt


def _advance(hist, q, nxt, y):
    move = (y != BLANK)[:, None]
    hist = [torch.where(move, torch.cat([h[:, 1:], y[:, None]], 1), h) for h in hist]
    return hist, torch.where(move[:, 0], nxt.gather(1, y[:, None])[:, 0], q)


def _decode(st, frames, S, B, k, compete, recombine):
    """The frame loop in float64: final histories, phrase states and totals."""
    H = S * B
    hist = [m.history(H) for m in st["models"]]
    q = torch.zeros(H, dtype=torch.int64, device="cuda")
    total = None if B == 1 else st["score0"].clone()
    name = torch.zeros(H, dtype=torch.int64, device="cuda")  # the emitted history, hashed
    for x in frames:
        key, fused, nxt = _keys(st, x, hist, q)
        if B == 1:
            if not compete:
                key[:, BLANK] = torch.where(x.argmax(1) == BLANK, math.inf, -math.inf)
            hist, q = _advance(hist, q, nxt, key.argmax(1))
            continue
        f, y = torch.topk(fused, k, dim=1)
        tot = (total[:, None] + f).reshape(S, B * k)
        y, who = y.reshape(S, B * k), torch.arange(H, device="cuda").repeat_interleave(k).reshape(S, B * k)
        moved = (name[who] ^ (y + 1) * 0x632BE59BD9B4E01) * 6364136223846793005 + 1442695
        hn = torch.where(y == BLANK, name[who], moved)
        if recombine:
            same = (hn[:, :, None] == hn[:, None, :]) & torch.isfinite(tot)[:, None, :]
            lead = same.int().argmax(2) == torch.arange(B * k, device="cuda")[None]
            merged = torch.logsumexp(torch.where(same, tot[:, None, :], -math.inf), 2)
            tot = torch.where(lead & torch.isfinite(tot), merged, -math.inf)
        tot, i = torch.sort(tot, dim=1, descending=True, stable=True)
        total, i = tot[:, :B].reshape(-1), i[:, :B]
        src, y, name = who.gather(1, i).reshape(-1), y.gather(1, i).reshape(-1), hn.gather(1, i).reshape(-1)
        hist, q = _advance([h[src] for h in hist], q[src], nxt[src], y)
    return hist, q, total


def exact(case, seed):
    kind, V = case["kind"], case["V"]
    st = prepare(case, seed)
    if kind == "project":
        out = st["A"].double() @ st["W"].double().t()
        return out if st["bias"] is None else out + st["bias"].double()
    if kind == "step":
        x = st["x"]
        key, fused, _ = _keys(st, x, st["hist"], st["boost"].long())
        if not case["compete"]:
            key[:, BLANK] = torch.where(x.argmax(1) == BLANK, math.inf, -math.inf)
        pick = torch.topk(key, case["k"], dim=1).indices
        out = dict(tokens=None, scores=fused.gather(1, pick), next_lm=None, next_boost=None)
        if case["fused"]:
            out["fused"] = fused
        return out
    S, B, T = case["S"], case["B"], case["T"]
    frames = st["x"]
    if kind == "projected":
        W, H = st["W"].double(), S * B
        frames = (st["A"][t * H:(t + 1) * H].double() @ W.t() + st["bias"].double() for t in range(T))
    elif B == 1 and not case["end"]:
        return None  # whole numbers only
    hist, q, total = _decode(st, frames, S, B, case["k"], case["compete"], case["recombine"])
    out = dict(tokens=None, lm=None, boost=None)
    if B > 1:
        out.update(parents=None, score=total)
    if kind == "projected":
        n = min(case["chunk"], T)
        last = T - (T % n or n)  # the last chunk's logits stand in the workspace's first rows
        x = torch.empty_like(st["x"], dtype=torch.float64)
        for a in ([last - n, last] if last >= n else [last]):
            rows = st["A"][a * H:min(a + n, T) * H].double() @ W.t() + st["bias"].double()
            x[:min(n, T - a)] = rows.reshape(-1, H, V)
        out["logits"] = x
        return out
    if case["end"]:
        term = sum(float(np.float32(a)) * m.rows(h)[:, V + 1] for m, a, h in zip(st["models"], st["alphas"], hist))
        out["end"] = term
        if B > 1:
            out["score"] = total + term
    return out
