"""GPU parity of greedy decoding where blank takes many frames: mode A passes
over the frames whose raw argmax is blank (64 at a time), and a greedy
hypothesis that emitted blank keeps its assembled rows.  Integer logits make
blank tie with lower and higher ids; blank sits at either end or inside the
vocabulary; frame counts lie around multiples of 64.  Tokens and final states
equal the oracle's, and those of a run that writes its fused rows (which scores
every frame), also on rows with infinities and NaN."""

import numpy as np
import pytest
import torch

import oracle
from oracle import traffic as checker
import paper_2609_14991_amd as F
from workloads import tiny_random_lm, tiny_random_phrases

pytestmark = pytest.mark.gpu


def _decode(glms, gtr, x, S, V, blank, mode, fused=False):
    n = len(glms)
    ls = torch.full((n, S), V, dtype=torch.int32, device="cuda")
    bs = torch.zeros((S,), dtype=torch.int32, device="cuda")
    out = F.run_lms(glms, [0.5, 0.25][:n], gtr, torch.from_numpy(x).to("cuda"), S, 1, 1, 0.5, blank, mode, ls, bs,
                    want_fused=fused)
    torch.cuda.synchronize()
    assert F.fusion_device_status() == 0
    return out["tokens"].cpu().numpy(), ls.cpu().numpy(), bs.cpu().numpy()


@pytest.mark.parametrize("V,n_lm", [(3, 1), (4, 1), (5, 2), (130, 1), (257, 2), (1001, 1), (1025, 1), (4097, 1)])
@pytest.mark.parametrize("mode", [F.FUSION_BLANK_AM, F.FUSION_BLANK_COMPETE])
def test_blank_frames(V, n_lm, mode):
    rng = np.random.default_rng(V * 7 + mode)
    for blank, T in [(0, 150), (V // 2, 65), (V - 1, 64)]:
        lms = [tiny_random_lm(rng, V, 3, n_sent=400, blank=blank) for _ in range(n_lm)]
        ph = tiny_random_phrases(rng, V, n=12, max_len=3, blank=blank, alphabet=min(V - 1, 12))
        glms, gtr = [F.ngram_load_arrays(m) for m in lms], F.boost_build_phrases(V, blank, ph)
        S = 5
        x = rng.integers(-3, 3, size=(T, S, V)).astype(np.float32)
        x[:, :, blank] = rng.integers(1, 4, size=(T, S))      # ties with the highest of the others, above, below
        x[:, 0, blank] = 9.0                                  # blank throughout
        x[:, 1, blank] = -9.0                                 # never
        tok, ls, bs = _decode(glms, gtr, x, S, V, blank, mode)
        r = oracle.run_lms([oracle.OracleLM(m) for m in lms], [0.5, 0.25][:n_lm], oracle.OracleTrie(V, blank, ph), x, S,
                           1, 1, 0.5, blank, mode, [[V] * S] * n_lm, [0] * S, threads=4)
        assert np.array_equal(tok, r["tokens"]), (blank, np.argwhere(tok != r["tokens"])[:3])
        assert np.array_equal(ls, np.asarray(r["lm_state"]).reshape(n_lm, S))
        assert np.array_equal(bs, r["boost_state"])
        x[3 % T, 2, :] = -np.inf
        x[5 % T, 3, blank] = -np.inf
        x[7 % T, 2, blank] = np.inf
        x[9 % T, 3, (blank + 1) % V] = np.inf
        x[11 % T, 4, [blank, (blank + 1) % V]] = np.inf
        x[13 % T, 4, (blank + 2) % V] = np.nan
        for a, b in zip(_decode(glms, gtr, x, S, V, blank, mode), _decode(glms, gtr, x, S, V, blank, mode, fused=True)):
            assert np.array_equal(a, b), blank


@pytest.mark.parametrize("V", [130, 1001, 2048])
def test_blank_frames_counted(V):
    """A run that counts its bytes goes through every frame: one that blank takes
    leaves nothing of its phrase state to the frames of the next state.  The count
    equals the independent one over the states visited."""
    rng = np.random.default_rng(V)
    S, T = 6, 150
    lm = tiny_random_lm(rng, V, 3, n_sent=400)
    ph = tiny_random_phrases(rng, V, n=30, max_len=5, alphabet=8)
    x = rng.normal(0.0, 1.0, size=(T, S, V)).astype(np.float32)
    x[:, :, 1:9] += 3.0
    x[:, :, 0] += np.where(rng.random((T, S)) < 0.5, 9.0, -9.0)
    ls = torch.full((S,), V, dtype=torch.int32, device="cuda")
    bs = torch.zeros((S,), dtype=torch.int32, device="cuda")
    count = torch.zeros(2, dtype=torch.int64, device="cuda")
    out = F.run(F.ngram_load_arrays(lm), F.boost_build_phrases(V, 0, ph), torch.from_numpy(x).to("cuda"), S, 1, 1, 0.5,
                2.0, 0, F.FUSION_BLANK_AM, ls, bs, traffic=count)
    torch.cuda.synchronize()
    assert F.fusion_device_status() == 0
    r = oracle.run(oracle.OracleLM(lm), oracle.OracleTrie(V, 0, ph), x, S, 1, 1, 0.5, 2.0, 0, F.FUSION_BLANK_AM,
                   [V] * S, [0] * S, threads=4)
    tok = out["tokens"].cpu().numpy()
    assert np.array_equal(tok, r["tokens"]), np.argwhere(tok != r["tokens"])[:3]
    assert np.array_equal(bs.cpu().numpy(), r["boost_state"])
    visits = checker.visited_states(oracle.OracleLM(lm), oracle.OracleTrie(V, 0, ph), V, 0, 1, r["tokens"])
    assert count.tolist() == list(checker.algorithmic_bytes(lm, ph, visits, T, beam=False))


@pytest.mark.parametrize("V,n_lm", [(3, 1), (130, 2), (1001, 1), (2048, 1), (8190, 1)])
@pytest.mark.parametrize("mode", [F.FUSION_BLANK_AM, F.FUSION_BLANK_COMPETE])
@pytest.mark.parametrize("fused", [False, True])
def test_rows_of_ff_bytes(V, n_lm, mode, fused):
    """A row of 0xFF bytes (the all-ones NaN in every token) offers no candidate: the
    frame goes to blank and the state stays, as if blank had won it outright."""
    rng = np.random.default_rng(V + mode)
    blank, S, T = 1, 3, 70
    lms = [tiny_random_lm(rng, V, 3, n_sent=400, blank=blank) for _ in range(n_lm)]
    ph = tiny_random_phrases(rng, V, n=12, max_len=3, blank=blank, alphabet=min(V - 1, 12))
    glms, gtr = [F.ngram_load_arrays(m) for m in lms], F.boost_build_phrases(V, blank, ph)
    x = rng.normal(0.0, 1.0, size=(T, S, V)).astype(np.float32)
    x[:, :, blank] += np.where(rng.random((T, S)) < 0.3, 9.0, -9.0)
    same = x.copy()
    for t, s in [(0, 0), (5, 1), (6, 1), (64, 2), (T - 1, 0)]:
        x.view(np.uint32)[t, s] = 0xFFFFFFFF
        same[t, s] = -50.0
        same[t, s, blank] = 50.0
    tok, ls, bs = _decode(glms, gtr, x, S, V, blank, mode, fused=fused)
    r = oracle.run_lms([oracle.OracleLM(m) for m in lms], [0.5, 0.25][:n_lm], oracle.OracleTrie(V, blank, ph), same, S,
                       1, 1, 0.5, blank, mode, [[V] * S] * n_lm, [0] * S, threads=4)
    assert np.array_equal(tok, r["tokens"]), np.argwhere(tok != r["tokens"])[:3]
    assert np.array_equal(ls, np.asarray(r["lm_state"]).reshape(n_lm, S))
    assert np.array_equal(bs, r["boost_state"])
