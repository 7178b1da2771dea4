"""GPU check that a beam's streams do not depend on how many share a call: S
streams, from fewer than the 8 blockIdx classes to a ragged number of them,
equal the same streams inside a call of 24, bit for bit (that call is a whole
multiple of the classes; its decode is checked against the oracle elsewhere)."""

import numpy as np
import pytest
import torch

import paper_2609_14991_amd as F
from workloads import tiny_random_lm, tiny_random_phrases

pytestmark = pytest.mark.gpu


def _decode(glm, gtr, x, S, B, k, V, flags):
    H = S * B
    ls = torch.full((1, H), V, dtype=torch.int32, device="cuda")
    bs = torch.zeros((H,), dtype=torch.int32, device="cuda")
    sc = torch.from_numpy(np.tile(np.array([0.0] + [-np.inf] * (B - 1)), S)).to("cuda")
    out = F.run_lms([glm], [0.5], gtr, x.contiguous(), S, B, k, 0.5, 0, F.FUSION_BLANK_COMPETE, ls, bs, sc,
                    recombine=flags)
    torch.cuda.synchronize()
    assert F.fusion_device_status() == 0
    return [t.cpu().reshape(-1, S, B) for t in (out["tokens"], out["parents"], ls, bs, sc)]


@pytest.mark.parametrize("V,B", [(200, 3), (700, 4), (1500, 8)])
@pytest.mark.parametrize("recombine", [False, True])
def test_streams_are_independent_of_the_launch(V, B, recombine):
    rng = np.random.default_rng(V + B)
    k = 4
    glm = F.ngram_load_arrays(tiny_random_lm(rng, V, 3, n_sent=2000))
    gtr = F.boost_build_phrases(V, 0, tiny_random_phrases(rng, V, n=30, max_len=4, alphabet=30))
    x = torch.from_numpy((rng.standard_normal((9, 24 * B, V)) * 2).astype(np.float32)).to("cuda")
    whole = _decode(glm, gtr, x, 24, B, k, V, recombine)
    for S in (1, 2, 7, 9, 23):
        part = _decode(glm, gtr, x[:, :S * B], S, B, k, V, recombine)
        for a, b in zip(part, whole):
            assert torch.equal(a, b[:, :S]), (V, B, S)


@pytest.mark.parametrize("V,B,k", [(1500, 32, 2), (4096, 17, 4), (700, 4, 4)])
def test_single_stream_beams_at_once(V, B, k):
    """Calls of one stream each on four HIP streams at a time: with the widest beams
    their slots are more than one XCD holds, and they must neither hold each other off nor
    change a result.  (All slots of the four calls fit the device.)"""
    rng = np.random.default_rng(V * B)
    glm = F.ngram_load_arrays(tiny_random_lm(rng, V, 3, n_sent=2000))
    gtr = F.boost_build_phrases(V, 0, tiny_random_phrases(rng, V, n=30, max_len=4, alphabet=30))
    T, n = 40, 4
    x = [torch.from_numpy((rng.standard_normal((T, B, V)) * 2).astype(np.float32)).to("cuda") for _ in range(n)]
    alone = [_decode(glm, gtr, a, 1, B, k, V, False) for a in x]
    sc0 = torch.tensor([0.0] + [-np.inf] * (B - 1), dtype=torch.float64, device="cuda")
    lanes = [torch.cuda.Stream() for _ in range(n)]
    state = [[torch.full((1, B), V, dtype=torch.int32, device="cuda"), torch.zeros(B, dtype=torch.int32, device="cuda"),
              sc0.clone(), torch.empty((T, B), dtype=torch.int32, device="cuda"),
              torch.empty((T, B), dtype=torch.int32, device="cuda")] for _ in range(n)]
    torch.cuda.synchronize()
    for a, (ls, bs, sc, tok, par), lane in zip(x, state, lanes):
        F.fusion_run_lms([glm], [0.5], gtr, a, T, 1, B, V, k, 0.5, 0, F.FUSION_BLANK_COMPETE, ls, bs, sc, tok, par,
                         stream=lane.cuda_stream)
    torch.cuda.synchronize()
    assert F.fusion_device_status() == 0
    for (ls, bs, sc, tok, par), want in zip(state, alone):
        for a, b in zip((tok, par, ls, bs, sc), want):
            assert torch.equal(a.cpu().reshape(-1), b.reshape(-1))
