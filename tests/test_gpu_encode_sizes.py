"""The encoder's lane layouts of small calls (one sub-vector per lane) and of large ones (sixteen channels per lane) store
the same bytes: a ragged batch encoded in one call, large enough for the second layout, against the same sequences encoded
one at a time with the first.  Lengths sit at the edges of the 8-token steps, 32- and 64-token workgroups.  The first layout is
compared with the oracle by the other encoder tests.  Every stored value is an fp16 or a code decided in fp64 (relative
differences of 1e-15 between the layouts' sums), so equality is exact."""
import numpy as np
import pytest

from paper_2505_18231_amd import synth
from tests import helpers

pytestmark = pytest.mark.gpu

LENS = [1, 7, 8, 63, 64, 65, 200, 385]
CASES = [  # (sub_dim, sign, rope, side_bits, group, page, capacity of the inputs, start)
    (4, False, False, 16, 0, 0, 385, 0),
    (4, False, True, 16, 64, 64, 385, 0),
    (8, False, False, 4, 64, 0, 385, 0),
    (8, True, True, 4, 64, 128, 385, 0),
    (8, True, False, 16, 128, 0, 640, 64),
    (4, False, False, 4, 0, 64, 385, 64),
    (8, False, False, 16, 0, 64, 385, 61),
]


@pytest.mark.parametrize("sub,sign,rope,side_bits,G,page,cap,start", CASES)
def test_one_large_call_equals_sequence_by_sequence(gpu_api, codebooks, sub, sign, rope, side_bits, G, page, cap,
                                                    start):
    import torch
    api = gpu_api
    B, H = len(LENS), 4
    if G == 128:
        start = 128  # a group's start
    print(f"case sub={sub} sign={sign} rope={rope} side_bits={side_bits} G={G} page={page} start={start}", flush=True)
    max_len = 1024
    g = torch.Generator(device="cuda").manual_seed(5)
    cb = torch.from_numpy(codebooks[sub].astype(np.float16)).cuda()
    cb = cb.abs() if sign else cb
    table = api.nsn_build_rope_table(synth.rope_inv_freq(5e5), max_len) if rope else None
    shape = api.make_shape(sub, H, H, max_len, G, page, sign_format=sign, rope_table=table, side_bits=side_bits)
    bt = torch.from_numpy(synth.shuffled_page_table(3, B, max_len // page)).cuda() if page else None
    k, v = (torch.randn((B, H, cap, 128), generator=g, device="cuda").half() for _ in range(2))
    k += 3.0
    n = torch.tensor(LENS, dtype=torch.int32, device="cuda")
    pos = torch.full((B,), start, dtype=torch.int32, device="cuda")
    freeze = start % 64 != 0 or (start > 0 and G == 0)
    large, single = (helpers.encode_layout(api, shape, n_seq, cap, freeze) for n_seq in (B, 1))
    assert large == 16 and single == sub               # the layout of large calls / the one of small calls

    def fresh():
        caches = api.alloc_cache(shape, B, block_table=bt), api.alloc_cache(shape, B, block_table=bt)
        for c in caches:       # stored means of the append mode
            if side_bits == 16:
                c.means.copy_((0.1 * torch.randn(c.means.shape, generator=torch.Generator().manual_seed(1))).half())
        return caches

    kc, vc = fresh()
    api.nsn_encode(shape, cb, k, v, pos, n, kc, vc, freeze_means=freeze)
    kr, vr = fresh()

    def part(c, b):
        if page:
            return api.CodedCache(c.codes, c.norms, c.means[b:b + 1], c.block_table[b:b + 1])
        return api.CodedCache(c.codes[b:b + 1], c.norms[b:b + 1], c.means[b:b + 1], None)

    for b in range(B):
        api.nsn_encode(shape, cb, k[b:b + 1].contiguous(), v[b:b + 1].contiguous(), pos[b:b + 1], n[b:b + 1], part(kr, b),
                       part(vr, b), freeze_means=freeze)
    torch.cuda.synchronize()
    for x, y in ((kc, kr), (vc, vr)):
        for name in ("codes", "norms", "means"):
            assert torch.equal(getattr(x, name), getattr(y, name)), name
        assert int((x.codes != 0).sum()) > 0


@pytest.mark.parametrize("sub,sign", [(4, False), (8, False), (8, True)])
def test_codewords_of_any_length(gpu_api, codebooks, select_variant, sub, sign):
    """Codewords a hundredth, down to a ten-thousandth, or a hundred times as long as the sub-vectors, and zero ones: the codes are those
    of the fp32 scan with its fp64 decision; and short codewords take the same path as the usual ones (the fp64 search of whole
    waves takes nine times as long; four is asked for)."""
    import time

    import torch
    api = gpu_api
    H, L = 8, 4096
    g = torch.Generator(device="cuda").manual_seed(7)
    k, v = (torch.randn((1, H, L, 128), generator=g, device="cuda").half() for _ in range(2))
    k[0, 0, 5] = 0.0
    k[0, 0, 6, 1:] = 0.0                                     # one channel: equal magnitudes after the rotation
    base = torch.from_numpy(codebooks[sub].astype(np.float32)).cuda()
    base = base.abs() if sign else base
    shape = api.make_shape(sub, H, H, L, 64, sign_format=sign)
    pos, n = torch.zeros(1, dtype=torch.int32, device="cuda"), torch.full((1,), L, dtype=torch.int32, device="cuda")
    ws = torch.empty(max(1, api.nsn_workspace_bytes(shape, api.NSN_OP_ENCODE, 1, L)), dtype=torch.uint8, device="cuda")
    took = {}
    for factor in (1.0, 0.01, 0.001, 0.0001, 100.0, 0.0):
        print(f"case sub={sub} sign={sign} factor={factor}", flush=True)
        cb = (base * factor).half()
        got = {}
        for impl in ("mfma", "valu"):
            select_variant("encode", impl)
            caches = api.alloc_cache(shape, 1), api.alloc_cache(shape, 1)
            api.nsn_encode(shape, cb, k, v, pos, n, *caches, workspace=ws)
            torch.cuda.synchronize()
            got[impl] = caches
        for x, y in zip(got["mfma"], got["valu"]):
            assert torch.equal(x.codes, y.codes) and torch.equal(x.norms, y.norms), factor
        select_variant("encode", "mfma")
        times = []
        for _ in range(5):
            start = time.perf_counter()
            for _ in range(5):
                api.nsn_encode(shape, cb, k, v, pos, n, *got["mfma"], workspace=ws)
            torch.cuda.synchronize()
            times.append(time.perf_counter() - start)
        took[factor] = min(times)
    print({f: f"{t / 5 * 1e6:.0f} us" for f, t in took.items()}, flush=True)
    assert took[0.01] < 4 * took[1.0]
