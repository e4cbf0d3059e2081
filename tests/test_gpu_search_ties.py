"""Codewords at equal distances: a codebook that holds rows twice or three times.  Every sub-vector nearest to such a row leaves
two candidates (in one group of eight codewords of the search or in two) or three, which fp64 distances settle for the lowest
index; codes are compared with an fp64 exhaustive search, and no later copy is ever taken."""
import numpy as np
import pytest

from oracle import nsn_oracle as O
from paper_2505_18231_amd import synth
from tests import helpers

pytestmark = pytest.mark.gpu

# copies (of row, at rows): two in one group of eight (rows 0..3 and 8..11 of a tile half), in neighbouring groups, in other tiles
PAIRS = [(0, [1]), (2, [11]), (4, [17]), (5, [21]), (33, [250]), (64, [70]), (255, [100]), (130, [131])]
MANY = [(0, [1, 2]), (8, [40, 200]), (77, [78, 79]), (99, [100])]


@pytest.mark.parametrize("sub,copies,tokens", [(4, PAIRS, 9), (8, PAIRS, 9), (4, PAIRS, 500), (8, PAIRS, 500), (4, MANY, 300), (8, MANY, 300)])
def test_equal_distances_go_to_the_lowest_index(gpu_api, codebooks, sub, copies, tokens):
    import torch
    api = gpu_api
    print(f"case sub={sub} tokens={tokens} copies={len(copies)}", flush=True)
    cb = codebooks[sub].astype(np.float16).astype(np.float64)
    lowest = np.arange(256)
    for row, at in copies:
        cb[at] = cb[row]
        lowest[[row, *at]] = min(row, *at)
    hkv, room = 16, 512
    shape = api.make_shape(sub, hkv, hkv, room, 0)
    kc, vc = api.alloc_cache(shape, 1), api.alloc_cache(shape, 1)
    k = np.stack([[synth.make_k(71, 0, h, tokens) for h in range(hkv)]])
    v = np.stack([[synth.make_v(71, 0, h, tokens) for h in range(hkv)]])
    n = torch.tensor([tokens], dtype=torch.int32, device="cuda")
    api.nsn_encode(shape, torch.from_numpy(cb.astype(np.float16)).cuda(), torch.from_numpy(k).cuda(), torch.from_numpy(v).cuda(),
                   torch.zeros_like(n), n, kc, vc)
    torch.cuda.synchronize()
    taken = 0
    for kind, dc, x in (("k", kc, k), ("v", vc, v)):
        h = helpers.HostCache(kind, 1, hkv, 128 // sub, room, 0)
        h.from_device(dc)
        for head in range(0, hkv, 5):
            got = h.unit_dict(0, head, tokens)
            ref = O.encode(x[0, head], cb, 0, given_b=got["b"], given_o=got["o"], return_debug=True)
            codes = got["codes"]
            assert np.array_equal(lowest[codes], codes), "a later copy of a codeword"
            # (the oracle's second best is at the same distance where a row has copies: nearest among distinct rows instead)
            y = ref["y"].reshape(tokens, 128 // sub, 1, sub)
            d = np.sort(((y - cb[np.unique(lowest)]) ** 2).sum(axis=3), axis=2)
            near_tie = d[:, :, 1] - d[:, :, 0] < 1e-6 * d[:, :, 1]
            assert np.all((codes == lowest[ref["codes"]]) | near_tie)
            taken += int(np.isin(codes, [lowest[row] for row, _ in copies]).sum())
    assert taken > 20, taken
