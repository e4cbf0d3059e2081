"""The ways a decode call is cut into workgroups give one result: splits chosen from the exact longest length (one for 136
units, five for 34), three forced splits, and the persistent instance, which a loose bound of the length selects for 136
units (the bound sizes the launch only).  Lengths sit at the edges of 64-token groups and of the 512 tokens up to which a
sequence is not split; 136 units (17 sequences with 8 kv heads of up to four query heads, or 4 of more) are no multiple of the
compute units.  The launches differ in the running maxima under which value weights are rounded to fp16: each weight
by 2^-11 at most, hence two results by 2^-10 < 1e-3 of the largest value."""
import math

import numpy as np
import pytest

from paper_2505_18231_amd import synth
from tests import helpers

pytestmark = pytest.mark.gpu

LENS = [0, 1, 63, 64, 65, 127, 511, 512, 513, 640, 1025, 300, 17, 256, 700, 129, 2049]
CASES = [  # (sub_dim, sign, rope, side_bits, group, page, kv heads, query heads per kv head, residual)
    (4, False, False, 16, 0, 64, 8, 4, False),
    (8, False, False, 4, 64, 0, 8, 3, True),
    (8, False, False, 16, 0, 64, 4, 8, True),
    (4, False, True, 16, 64, 64, 8, 1, True),
    (8, True, False, 16, 64, 64, 8, 4, True),
    (8, True, False, 4, 0, 0, 8, 2, False),
    (8, True, True, 4, 64, 64, 8, 4, True),
    (8, True, True, 16, 0, 0, 4, 6, False),
    (4, False, False, 16, 0, 64, 2, 4, True),
    (8, True, True, 4, 64, 0, 2, 4, False),
]


@pytest.mark.parametrize("sub,sign,rope,side_bits,G,page,H,r,residual", CASES)
def test_every_cut_gives_the_same_result(gpu_api, codebooks, sub, sign, rope, side_bits, G, page, H, r,
                                              residual):
    import torch
    api = gpu_api
    B, room, scale = len(LENS), 16384, 1.0 / math.sqrt(128)
    print(f"case sub={sub} sign={sign} rope={rope} side_bits={side_bits} G={G} page={page} H={H} r={r} residual={residual}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(6)
    cb = torch.from_numpy(codebooks[sub].astype(np.float16)).cuda()
    cb = cb.abs() if sign else cb
    table = api.nsn_build_rope_table(synth.rope_inv_freq(5e5), room) if rope else None
    shape = api.make_shape(sub, H * r, H, room, G, page, sign_format=sign, rope_table=table, side_bits=side_bits)
    bt = torch.from_numpy(synth.shuffled_page_table(3, B, room // page)).cuda() if page else None
    kc, vc = api.alloc_cache(shape, B, block_table=bt), api.alloc_cache(shape, B, block_table=bt)
    n = torch.tensor(LENS, dtype=torch.int32, device="cuda")
    k, v = (torch.randn((B, H, max(LENS), 128), generator=g, device="cuda").half() for _ in range(2))
    api.nsn_encode(shape, cb, k + 1.0, v, torch.zeros_like(n), n, kc, vc)
    q = torch.randn((B, H * r, 128), generator=g, device="cuda").half()
    rows = [torch.randn((B, H, 64, 128), generator=g, device="cuda").half() for _ in range(2)]
    res_lens = torch.arange(B, dtype=torch.int32, device="cuda") * 4 % 65
    outs = []
    few = B * H < 64
    for bound, n_splits, cut in ((max(LENS), 0, 5 if few else 1), (max(LENS), 3, 3), (room, 0, 7 if few else 0)):
        assert helpers.decode_splits(api, shape, B, bound, n_splits) == cut
        if residual:
            o = api.nsn_decode_attention_residual(shape, cb, q, kc, vc, n, bound, *rows, res_lens, scale, n_splits)
        else:
            o = api.nsn_decode_attention(shape, cb, q, kc, vc, n, bound, scale, n_splits)
        torch.cuda.synchronize()
        outs.append(o.cpu().numpy().astype(np.float64))
    assert np.all(np.isfinite(outs[0])) and (residual or np.all(outs[0][0] == 0.0))
    for o in outs[1:]:
        err = max(helpers.max_rel_err(outs[0][b], o[b]) for b in range(B) if residual or LENS[b])
        print(f"  largest difference {err:.3e}", flush=True)
        assert err < 1e-3, err
