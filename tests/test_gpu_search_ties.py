"""Codewords at equal distances: a codebook that holds rows twice or three times.  Every sub-vector nearest to such a row leaves
two candidates (in one group of eight codewords of the search or in two) or three, which fp64 distances settle for the lowest
index; codes are compared with an fp64 exhaustive search, and no later copy is ever taken.  In the encoder and in K-Means, whose
instances of the search hold other operands (codewords with a low part)."""
import numpy as np
import pytest

from oracle import nsn_oracle as O
from paper_2505_18231_amd import synth
from tests import helpers

pytestmark = pytest.mark.gpu

# copies (of row, at rows): two in one group of eight (codewords lie in order), in neighbouring groups, in other tiles
PAIRS = [(0, [1]), (2, [11]), (4, [17]), (5, [21]), (33, [250]), (64, [70]), (255, [100]), (130, [131])]
MANY = [(0, [1, 2]), (8, [40, 200]), (77, [78, 79]), (99, [100])]
# 32 and 33 equal rows: the most that the lists settle, and one more
EDGE = [(3, list(range(60, 91))), (100, list(range(120, 152)))]


@pytest.mark.parametrize("sub,copies,tokens", [(4, PAIRS, 9), (8, PAIRS, 9), (4, PAIRS, 500), (8, PAIRS, 500), (4, MANY, 300), (8, MANY, 300),
                                               (4, EDGE, 100), (8, EDGE, 100)])
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


@pytest.mark.parametrize("sub,copies,n", [(4, PAIRS, 4000), (8, PAIRS, 4000), (4, PAIRS, 300), (8, PAIRS, 1 << 16), (4, MANY, 4000), (8, MANY, 4000),
                                          (8, MANY, 1 << 16), (4, EDGE, 4000), (8, EDGE, 4000)])
def test_kmeans_gives_all_members_to_the_lowest_copy(gpu_api, sub, copies, n):
    """One iteration from first samples that hold rows twice or more: the later copies get no member and stay what they were, the
    lowest one becomes the mean of all."""
    import torch
    print(f"case sub={sub} n={n} copies={len(copies)}", flush=True)
    samples = synth.codebook_samples(63, n, sub)
    later = []
    for row, at in copies:
        samples[at] = samples[row]
        later += [k for k in (row, *at) if k != min(row, *at)]
    c = samples[:256].astype(np.float64)
    near = np.empty(n, np.int64)
    for t in range(0, n, 4096):  # (equal rows have equal distances: the first one is taken)
        near[t:t + 4096] = ((samples[t:t + 4096, None, :].astype(np.float64) - c[None]) ** 2).sum(axis=2).argmin(axis=1)
    ref = np.stack([samples[near == k].astype(np.float64).mean(axis=0) if (near == k).any() else c[k] for k in range(256)])
    cb, _ = gpu_api.nsn_build_codebook(torch.from_numpy(samples).cuda(), 256, 1)
    got = cb.cpu().numpy()
    assert np.array_equal(got[later], samples[later].astype(np.float16)), "a later copy got members"
    diff = np.abs(got.view(np.int16).astype(np.int32) - ref.astype(np.float16).view(np.int16).astype(np.int32))
    print(f"  {(diff != 0).sum()} of {diff.size} fp16 entries differ, max {diff.max()} ulp", flush=True)
    # both are single fp16 roundings of fp64 centroids that differ only by summation order
    assert diff.max() <= 1 and (diff == 0).mean() > 0.999
