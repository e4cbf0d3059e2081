"""Splits of more than 2^25 tokens: the descriptors through which contiguous caches are read have 32-bit offsets and move on
inside the main loop.  One split of the whole sequence against 64 splits of half a million tokens each, which never do.

Only the last tokens carry values and scores other than zero, so the sums stay exact far enough: the fp32 sums of the others'
weights (ones) are whole numbers below 2^24 in every lane, and what is left is the rounding of one softmax either way."""
import math

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("group", [0, 64])
def test_one_split_of_more_tokens_than_an_offset_reaches(gpu_api, group):
    api = gpu_api
    tail, L = 4096 + 17, (1 << 25) + 8192 + 17
    max_len = (L + 63) // 64 * 64
    shape = api.make_shape(8, 4, 1, max_len, group)
    g = torch.Generator(device="cuda").manual_seed(5)
    cb = torch.randn((256, 8), generator=g, device="cuda").half()
    caches = []
    for _ in range(2):
        c = api.alloc_cache(shape, 1)
        c.codes.random_(0, 256, generator=g)
        far = c.norms.view(-1, 2)[L - tail:L]
        far.copy_(torch.rand(far.shape, generator=g, device="cuda").half() + 0.5)
        c.means.copy_(torch.randn(c.means.shape, generator=g, device="cuda", dtype=torch.float16))
        caches.append(c)
    q = torch.randn((1, 4, 128), generator=g, device="cuda").half()
    lens = torch.tensor([L], dtype=torch.int32, device="cuda")
    out = [api.nsn_decode_attention(shape, cb, q, *caches, lens, L, 1.0 / math.sqrt(128), n_splits=n) for n in (1, 64)]
    torch.cuda.synchronize()
    err = float((out[0] - out[1]).abs().max() / out[1].abs().max())
    print(f"group {group}: max rel err {err:.2e}", flush=True)
    assert err < 2e-3, err
