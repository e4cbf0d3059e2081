"""Codewords that hold a NaN are never taken while any other codeword is there, whatever the NaN's sign: no distance to them is
a number, as in an exhaustive search that starts from infinity.  (The sign counts because the search lists its candidates by the sign
bit of a difference: a NaN that a host's 0/0 gives has it set.)"""
import numpy as np
import pytest

from oracle import nsn_oracle as O
from paper_2505_18231_amd import synth
from tests import helpers

pytestmark = pytest.mark.gpu

NAN16 = {False: 0x7E00, True: 0xFE00}
NAN32 = {False: 0x7FC00000, True: 0xFFC00000}
# in one group of eight codewords of the search ahead of the nearest ones and behind them, in other groups, and most of a group
ROWS = [0, 19, 20, 63, 100, 130, 250, 232, 233, 234, 235, 240]


@pytest.mark.parametrize("negative", [True, False])
@pytest.mark.parametrize("sub,sign", [(4, False), (8, False), (8, True)])
def test_a_codeword_that_is_not_a_number_is_not_taken(gpu_api, codebooks, sub, sign, negative):
    import torch
    api = gpu_api
    print(f"case sub={sub} sign={sign} negative={negative}", flush=True)
    hkv, tokens = 16, 200
    cb = np.abs(codebooks[sub]) if sign else codebooks[sub]
    cb16 = cb.astype(np.float16)
    cb16.view(np.uint16)[ROWS, np.arange(len(ROWS)) % sub] = NAN16[negative]   # one element of the row
    far = cb16.astype(np.float64)
    far[ROWS] = 6.0e4                                                        # the same choice: never the nearest
    shape = api.make_shape(sub, hkv, hkv, 256, 0, sign_format=sign)
    kc, vc = api.alloc_cache(shape, 1), api.alloc_cache(shape, 1)
    k = np.stack([[synth.make_k(73, 0, h, tokens) for h in range(hkv)]])
    v = np.stack([[synth.make_v(73, 0, h, tokens) for h in range(hkv)]])
    n = torch.tensor([tokens], dtype=torch.int32, device="cuda")
    api.nsn_encode(shape, torch.from_numpy(cb16).cuda(), torch.from_numpy(k).cuda(), torch.from_numpy(v).cuda(),
                   torch.zeros_like(n), n, kc, vc)
    torch.cuda.synchronize()
    J = 128 // sub
    for kind, dc, x in (("k", kc, k), ("v", vc, v)):
        h = helpers.HostCache(kind, 1, hkv, 2 * J if sign else J, 256, 0, layout="legacy" if sign else "tiled")
        h.from_device(dc)
        for head in range(hkv):
            got = h.unit_dict(0, head, tokens)
            codes = got["codes"][:, :J]
            assert not np.isin(codes, ROWS).any(), np.unique(codes[np.isin(codes, ROWS)])
            assert np.isfinite(got["a"].astype(np.float64)).all()
            if head % 5 == 0:
                given = dict(given_b=got["b"], given_o=got["o"], return_debug=True)
                ref = O.encode(x[0, head], far, 0, sign_format=True, **given) if sign else O.encode(x[0, head], far, 0, **given)
                y = ref["y"].reshape(tokens, J, 1, sub)
                y = np.abs(y) if sign else y
                d = ((y - far) ** 2).sum(axis=3)
                two = np.sort(d, axis=2)[:, :, :2]
                near_tie = two[:, :, 1] - two[:, :, 0] < 1e-6 * two[:, :, 1]
                assert np.all((codes == d.argmin(axis=2)) | near_tie)


@pytest.mark.parametrize("negative", [True, False])
@pytest.mark.parametrize("sub", [4, 8])
def test_kmeans_takes_no_codeword_that_became_not_a_number(gpu_api, sub, negative):
    """A sample that holds a NaN belongs to the first codeword, which is not a number from then on: every later iteration deals all
    other samples out to the other codewords."""
    import torch
    print(f"case sub={sub} negative={negative}", flush=True)
    samples = synth.codebook_samples(58, 4013, sub)
    samples.view(np.uint32)[700, 1] = NAN32[negative]
    finite = np.arange(len(samples)) != 700
    x, c = samples[finite].astype(np.float64), samples[:256].astype(np.float64)
    for step in range(3):
        d = ((x[:, None, :] - c[None]) ** 2).sum(axis=2)
        if step:
            d[:, 0] = np.inf
        near = d.argmin(axis=1)
        for r in range(1, 256):
            if (near == r).any():
                c[r] = x[near == r].mean(axis=0)
    cb, _ = gpu_api.nsn_build_codebook(torch.from_numpy(samples).cuda(), 256, 3)
    got, ref = cb.cpu().numpy(), c.astype(np.float16)
    assert np.isnan(got[0, 1])
    diff = np.abs(got[1:].view(np.int16).astype(np.int32) - ref[1:].view(np.int16).astype(np.int32))
    print(f"  {(diff != 0).sum()} of {diff.size} entries differ, max {diff.max()} ulp", flush=True)
    # single fp16 roundings of fp64 centroids that differ only by summation order (1e-13 before the rounding)
    assert diff.max() <= 1 and (diff == 0).mean() > 0.999
