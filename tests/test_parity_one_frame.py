"""GPU parity of greedy decoding one frame per call: a call of one frame runs as
a step with its states in place, and a stream fed frame by frame must give the
tokens, states and fused rows of one call over all frames, and the oracle's
tokens and states.  Also where the frame has no ordinary answer: states out of
range (blank, states unchanged, status set), rows of infinities, NaN and 0xFF
bytes."""

import numpy as np
import pytest
import torch

import oracle
import paper_2609_14991_amd as F
from workloads import tiny_random_lm, tiny_random_phrases

pytestmark = pytest.mark.gpu

ALPHAS = [0.5, 0.25]


def _decode(glms, gtr, x, blank, mode, chunk, ls, bs, fused, count=False):
    T, S, V = x.shape
    ls = torch.from_numpy(np.ascontiguousarray(ls, dtype=np.int32)).to("cuda")
    bs = None if gtr is None else torch.from_numpy(np.ascontiguousarray(bs, dtype=np.int32)).to("cuda")
    tok = torch.full((T, S), -7, dtype=torch.int32, device="cuda")
    row = torch.full((T, S, V), 7.0, device="cuda") if fused else None
    n = torch.zeros(2, dtype=torch.int64, device="cuda") if count else None
    for t in range(0, T, chunk):
        c = min(chunk, T - t)
        F.fusion_run_lms(glms, ALPHAS[:len(glms)], gtr, x[t:t + c], c, S, 1, V, 1, 0.5, blank, mode, ls, bs, None,
                         tok[t:t + c], None, None if row is None else row[t:t + c], n)
    torch.cuda.synchronize()
    out = [tok.cpu().numpy(), ls.cpu().numpy()] + ([] if bs is None else [bs.cpu().numpy()])
    return out + ([] if row is None else [row.cpu().numpy().view(np.uint32)]), F.fusion_device_status()


def _same(a, b):
    assert a[1] == b[1]
    for u, v in zip(a[0], b[0]):
        assert np.array_equal(u, v), np.argwhere(u != v)[:3]


@pytest.mark.parametrize("V,n_lm", [(2, 1), (5, 2), (128, 1), (257, 2), (1001, 1), (1024, 1), (4094, 2), (4096, 1),
                                    (8190, 1)])
@pytest.mark.parametrize("mode", [F.FUSION_BLANK_AM, F.FUSION_BLANK_COMPETE])
@pytest.mark.parametrize("trie", [True, False])
def test_one_frame_calls(V, n_lm, mode, trie):
    rng = np.random.default_rng(V * 5 + mode)
    blank, S, T = V // 3, 5, 24
    lms = [tiny_random_lm(rng, V, 4, n_sent=400, blank=blank) for _ in range(n_lm)]
    ph = tiny_random_phrases(rng, V, n=12, max_len=3, blank=blank, alphabet=min(V - 1, 12))
    glms = [F.ngram_load_arrays(m) for m in lms]
    gtr = F.boost_build_phrases(V, blank, ph) if trie else None
    x = rng.normal(0.0, 1.0, size=(T, S, V)).astype(np.float32)
    x[:, :, :min(V, 12)] += 3.0
    x[:, :, blank] += np.where(rng.random((T, S)) < 0.4, 9.0, -9.0)
    start, root = np.full((n_lm, S), V), np.zeros(S)
    xd = torch.from_numpy(x).to("cuda")
    one = _decode(glms, gtr, xd, blank, mode, 1, start, root, False)
    r = oracle.run_lms([oracle.OracleLM(m) for m in lms], ALPHAS[:n_lm], oracle.OracleTrie(V, blank, ph) if trie else None,
                       x, S, 1, 1, 0.5, blank, mode, [[V] * S] * n_lm, [0] * S, threads=4)
    assert one[1] == 0
    assert np.array_equal(one[0][0], r["tokens"])
    assert np.array_equal(one[0][1], np.asarray(r["lm_state"]).reshape(n_lm, S))
    if trie:
        assert np.array_equal(one[0][2], r["boost_state"])
    _same(one, _decode(glms, gtr, xd, blank, mode, T, start, root, False))
    _same(one, _decode(glms, gtr, xd, blank, mode, 1, start, root, False, count=True))
    # rows off 16 bytes, with the fused rows
    off = torch.zeros(xd.numel() + 1, device="cuda")[1:].view(T, S, V).copy_(xd)
    _same(_decode(glms, gtr, off, blank, mode, 1, start, root, True),
          _decode(glms, gtr, xd, blank, mode, T, start, root, True))
    # states out of range, and rows without an ordinary answer
    start[0, 1], start[-1, 2] = blank, 1 << 30
    root[3] = -5
    x[2, 0] = -np.inf
    x[3, 0, blank] = -np.inf
    x[4, 4, blank] = np.inf
    x[5, 4, (blank + 1) % V] = np.nan
    x[6, 0, blank] = np.nan
    x.view(np.uint32)[7, [0, 4]] = 0xFFFFFFFF
    x[8, 0] = np.nan
    xd = torch.from_numpy(x).to("cuda")
    one = _decode(glms, gtr, xd, blank, mode, 1, start, root, False)
    assert one[1] == F.FUSION_STATUS_BAD_LM_STATE | (F.FUSION_STATUS_BAD_BOOST_STATE if trie else 0)
    _same(one, _decode(glms, gtr, xd, blank, mode, T, start, root, False))
    assert (one[0][0][:, 1] == blank).all() and one[0][1][0, 1] == blank and one[0][1][-1, 2] == 1 << 30
    assert (one[0][0][7, [0, 4]] == blank).all()
