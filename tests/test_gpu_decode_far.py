"""Splits of more than 2^26 tokens: the descriptors through which contiguous caches are read span 2^26 of them, and they and the
Shift vectors' base move on every 2^25 inside the main loop (twice here; behind the first span an unmoved descriptor reads zeros).
One split of the whole sequence against 64 splits of a million tokens each, which never move.  By format: 16 and 32 bytes per
token (a span of 2^31 bytes), 4-bit side information and pages (block numbers: only the Shift vectors' base moves), sign codes
and keys before the rotary embedding (the legacy layout).  The persistent instance moves by the same code, but its runs are that
long only from 2^33 tokens on.

Only the last tokens carry values and scores other than zero, so the sums stay exact far enough: the fp32 sums of the others'
weights (ones) are whole numbers below 2^24 in every lane, and what is left is the rounding of one softmax either way."""
import math

import pytest

torch = pytest.importorskip("torch")
from paper_2505_18231_amd import synth  # noqa: E402

pytestmark = pytest.mark.gpu

# sub_dim, group, side_bits, page, sign, rope
CASES = [(8, 0, 16, 0, False, False), (8, 64, 16, 0, False, False), (4, 192, 16, 0, False, False), (4, 0, 4, 0, False, False),
         (8, 64, 16, 4096, False, False), (8, 64, 16, 0, True, False), (8, 0, 4, 0, True, False), (8, 64, 16, 0, False, True)]


@pytest.mark.parametrize("sub,group,side_bits,page,sign,rope", CASES)
def test_one_split_of_more_tokens_than_a_descriptor_spans(gpu_api, sub, group, side_bits, page, sign, rope):
    api = gpu_api
    print(f"case sub={sub} group={group} side_bits={side_bits} page={page} sign={sign} rope={rope}", flush=True)
    tail, L = 4096 + 17, (1 << 26) + 8192 + 17
    max_len = (L + 4095) // 4096 * 4096
    max_len += -max_len % group if group == 192 else 0
    table = api.nsn_build_rope_table(synth.rope_inv_freq(5e5), max_len) if rope else None
    shape = api.make_shape(sub, 4, 1, max_len, group, page, sign_format=sign, rope_table=table, side_bits=side_bits)
    g = torch.Generator(device="cuda").manual_seed(5)
    cb = torch.randn((256, sub), generator=g, device="cuda").half()
    cb = cb.abs() if sign else cb
    pages = torch.arange(max_len // page - 1, -1, -1, dtype=torch.int32, device="cuda").view(1, -1) if page else None
    caches = []
    for _ in range(2):
        c = api.alloc_cache(shape, 1, block_table=pages)
        c.codes.random_(0, 256, generator=g)
        if side_bits == 4:  # 64 a', 64 four-bit codes of b, (min, step) of b
            far = c.norms.view(-1, 164)[(L - tail) // 64:(L + 63) // 64]
            far[:, :128] = (torch.rand((len(far), 64), generator=g, device="cuda").half() + 0.5).view(torch.uint8)
            far[:, 128:160].random_(0, 256, generator=g)
            far[:, 160:] = torch.tensor([0.5, 0.0625], device="cuda").half().view(torch.uint8)
            c.means[..., :64].random_(0, 256, generator=g)
            c.means[..., 64:] = torch.tensor([-1.0, 0.125] * 4, device="cuda").half().view(torch.uint8)
        else:
            far = c.norms.view(-1, 2)
            at = torch.arange(L - tail, L, device="cuda")
            if page:  # page p of the sequence is the buffer's (n - 1 - p)-th
                at = (max_len // page - 1 - at // page) * page + at % page
            far[at] = torch.rand((tail, 2), generator=g, device="cuda").half() + 0.5
            c.means.copy_(torch.randn(c.means.shape, generator=g, device="cuda", dtype=torch.float16))
        caches.append(c)
    q = torch.randn((1, 4, 128), generator=g, device="cuda").half()
    lens = torch.tensor([L], dtype=torch.int32, device="cuda")
    out = [api.nsn_decode_attention(shape, cb, q, *caches, lens, L, 1.0 / math.sqrt(128), n_splits=n) for n in (1, 64)]
    torch.cuda.synchronize()
    err = float((out[0] - out[1]).abs().max() / out[1].abs().max())
    print(f"  max rel err {err:.2e}", flush=True)
    assert float(out[1].abs().max()) > 0
    assert err < 2e-3, err
