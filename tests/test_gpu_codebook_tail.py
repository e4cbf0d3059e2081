"""Ordered sums (fine-tuning, and K-Means of samples that fixed-point sums do not hold) of sample counts that are no multiple of the
runs of sixteen: up to fifteen samples behind the last whole run, the last of their chains' order, and counts that leave most
chains without samples."""
import numpy as np
import pytest

from oracle import nsn_oracle as O
from paper_2505_18231_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sub,n", [(4, 8193), (8, 8207), (4, 16389), (8, 301), (4, 257)])
def test_finetune_of_any_sample_count(gpu_api, sub, n):
    import torch
    print(f"case sub={sub} n={n}", flush=True)
    samples = synth.codebook_samples(61, n, sub)
    start, _, _ = O.build_codebook(samples, 256, 2)
    ref, hist, ref_final = O.finetune_codebook(samples, start, 3, 64.0)
    x = torch.from_numpy(samples).cuda()
    cb, cos0, cos1 = gpu_api.nsn_finetune_codebook(x, torch.from_numpy(start.astype(np.float16)).cuda(), 3, 64.0)
    got = cb.cpu().numpy()
    diff = np.abs(got.view(np.int16).astype(np.int32) - ref.astype(np.float16).view(np.int16).astype(np.int32))
    print(f"  {(diff != 0).sum()} of {diff.size} fp16 entries differ, max {diff.max()} ulp", flush=True)
    # (the fp64 sums differ from the oracle's in the order of addition: 1e-13 before the entries are rounded to fp16)
    assert diff.max() <= 1 and (diff == 0).mean() > 0.995
    assert abs(cos0 - hist[0]) < 1e-12 and abs(cos1 - ref_final) < 1e-9 + 1e-5 * (diff.max() > 0)


@pytest.mark.parametrize("finite", [True, False])
@pytest.mark.parametrize("sub,n", [(4, 4001), (8, 4013), (4, 301), (8, 303), (8, 257)])
def test_kmeans_of_any_sample_count_with_ordered_sums(gpu_api, sub, n, finite):
    """A sample 2^60 times the others, or an infinity: the centroids of all others are means over every member, those behind the
    last whole run among them (as many of the last samples as there are behind it are made members of one codeword, which a lost or
    doubled one would move by far more than a rounding)."""
    import torch
    print(f"case sub={sub} n={n} finite={finite}", flush=True)
    samples = synth.codebook_samples(62, n, sub)
    tail = n % 16
    samples[n - tail:] = samples[100] + np.float32(0.02) * (1 + np.arange(tail, dtype=np.float32)[:, None])
    samples[7, 1] = 2.0 ** 60 if finite else np.inf
    x, c = samples.astype(np.float64), samples[:256].astype(np.float64)
    for _ in range(2 if finite else 1):  # (an infinite centroid has no finite distance to anything: one iteration)
        with np.errstate(invalid="ignore"):
            d = ((x[:, None, :] - c[None]) ** 2).sum(axis=2)
        near = np.where(np.isnan(d) | ~np.isfinite(d), np.inf, d).argmin(axis=1)
        c = np.stack([x[near == k].mean(axis=0) if (near == k).any() else c[k] for k in range(256)])
    cb, _ = gpu_api.nsn_build_codebook(torch.from_numpy(samples).cuda(), 256, 2 if finite else 1)
    rows = np.abs(c).max(axis=1) < 100
    assert rows.sum() >= 254 and np.unique(near[n - tail:]).size < tail or tail == 1
    got, ref = cb.cpu().numpy()[rows], c[rows].astype(np.float16)
    # both are single fp16 roundings of fp64 centroids that differ only by summation order
    diff = np.abs(got.view(np.int16).astype(np.int32) - ref.view(np.int16).astype(np.int32))
    print(f"  {(diff != 0).sum()} of {diff.size} fp16 entries differ, max {diff.max()} ulp", flush=True)
    assert diff.max() <= 1 and (diff == 0).mean() > 0.999
