"""The encoder's instances for three workgroups to a compute unit store the same bytes as those for two: a ragged batch of nine
sequences (2160 workgroups of 64 tokens) against three calls of three sequences each (720).  Both take the sixteen-channel layout;
lengths sit at the edges of its 8-token steps and of the workgroups."""
import numpy as np
import pytest

from paper_2505_18231_amd import synth
from tests import helpers

pytestmark = pytest.mark.gpu

CAP = 320
LENS = [1, 7, 320, 8, 65, 319, 63, 128, 257]
# sub_dim, sign, rope, group, side_bits, page, start
CASES = [(4, False, False, 0, 16, 0, 0), (4, False, True, 128, 16, 128, 61), (4, False, False, 64, 4, 64, 0),
         (8, False, False, 0, 16, 64, 30), (8, False, True, 0, 4, 0, 64), (8, True, False, 256, 16, 256, 7), (8, True, True, 64, 4, 0, 0)]


@pytest.mark.parametrize("sub,sign,rope,G,side_bits,page,start", CASES)
def test_large_call_equals_its_parts(gpu_api, codebooks, sub, sign, rope, G, side_bits, page, start):
    import torch
    api = gpu_api
    print(f"case sub={sub} sign={sign} rope={rope} G={G} side_bits={side_bits} page={page} start={start}", flush=True)
    B, H, max_len = len(LENS), 24, 1024
    g = torch.Generator(device="cuda").manual_seed(21)
    cb = torch.from_numpy(codebooks[sub].astype(np.float16)).cuda()
    if sign:
        cb = cb.abs()
    table = api.nsn_build_rope_table(synth.rope_inv_freq(5e5), max_len) if rope else None
    shape = api.make_shape(sub, H, H, max_len, G, page, sign_format=sign, rope_table=table, side_bits=side_bits)
    bt = torch.from_numpy(synth.shuffled_page_table(3, B, max_len // page)).cuda() if page else None
    k, v = (torch.randn((B, H, CAP, 128), generator=g, device="cuda").half() for _ in range(2))
    k += 3.0
    n = torch.tensor(LENS, dtype=torch.int32, device="cuda")
    pos = torch.full((B,), start, dtype=torch.int32, device="cuda")
    freeze = start > 0
    assert [helpers.encode_launch_form(api, shape, n_seq, CAP, freeze) for n_seq in (B, 3)] == [(16, 64, 3), (16, 64, 2)]

    def fresh():
        caches = api.alloc_cache(shape, B, block_table=bt), api.alloc_cache(shape, B, block_table=bt)
        for c in caches:
            if side_bits == 16:
                c.means.copy_((0.1 * torch.randn(c.means.shape, generator=torch.Generator().manual_seed(1))).half())
        return caches

    kc, vc = fresh()
    api.nsn_encode(shape, cb, k, v, pos, n, kc, vc, freeze_means=freeze)
    kr, vr = fresh()

    def part(c, at):
        if page:
            return api.CodedCache(c.codes, c.norms, c.means[at], c.block_table[at])
        return api.CodedCache(c.codes[at], c.norms[at], c.means[at], None)

    for b in range(0, B, 3):
        at = slice(b, b + 3)
        api.nsn_encode(shape, cb, k[at], v[at], pos[at], n[at], part(kr, at), part(vr, at), freeze_means=freeze)
    torch.cuda.synchronize()
    for x, y in ((kc, kr), (vc, vr)):
        for name in ("codes", "norms", "means"):
            assert torch.equal(getattr(x, name), getattr(y, name)), name
        assert int((x.codes != 0).sum()) > 0
