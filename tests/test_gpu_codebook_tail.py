"""Fine-tuning of sample counts that are no multiple of the runs of sixteen: up to fifteen samples behind the last whole run, the last
of their chains' order, and counts that leave most chains without samples."""
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
