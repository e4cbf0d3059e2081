"""The search's form for three workgroups to a compute unit where it can go wrong: equal codewords at the edges of its groups (4-dim:
seven and nine to sixteen codewords, 7 and 8 of them in both groups), codewords that hold a NaN or an infinity, very short, very long
and zero ones (fp16 rows below the smallest normal number; sub-vectors out of range, which take the fp64 search), tokens of zeros,
with a single channel, with a NaN or an infinity.  One sequence of 640 workgroups against the same tokens in four calls, whose
instances (two workgroups) are compared with the oracle by the other tests, and, where no codeword is a NaN or infinite, against
the fp32 scan.  Equality is exact: codes are decided in fp64."""
import numpy as np
import pytest

from paper_2505_18231_amd import synth
from tests import helpers

pytestmark = pytest.mark.gpu

H, L, PART = 8, 2560, 640
COPIES = [(7, [8]), (22, [23]), (24, [25]), (39, [40, 41]), (54, [55, 200]), (72, [71]), (87, [88, 151, 152]), (103, [111]), (127, [128]),
          (135, [143, 144]), (6, [15]), (247, [248]), (255, [231])]
EDGE = [(3, list(range(60, 91))), (100, list(range(120, 152)))]  # 32 and 33 equal rows
BOOKS = ["copies", "edge", "nan", "nan with its sign set", "inf", "0.01", "0.0001", "100", "0"]


def _book(cb, kind, sub):
    cb16 = cb.astype(np.float16)
    if kind in ("copies", "edge"):
        for row, at in COPIES if kind == "copies" else EDGE:
            cb16[at] = cb16[row]
    elif kind.startswith("nan"):
        rows = [0, 7, 8, 9, 23, 24, 100, 232, 233, 234, 235, 240]
        cb16.view(np.uint16)[rows, np.arange(len(rows)) % sub] = 0xFE00 if "sign" in kind else 0x7E00
    elif kind == "inf":
        cb16[[7, 24, 130], [0, 1, 2]] = [np.inf, -np.inf, np.inf]
    else:
        cb16 = (cb * float(kind)).astype(np.float16)
    return cb16


@pytest.mark.parametrize("kind", BOOKS)
@pytest.mark.parametrize("sub,sign,rope", [(4, False, False), (4, False, True), (8, False, False), (8, True, True)])
def test_hard_codebooks_and_tokens(gpu_api, codebooks, select_variant, sub, sign, rope, kind):
    import torch
    api = gpu_api
    print(f"case sub={sub} sign={sign} rope={rope} codebook={kind}", flush=True)
    cb16 = _book(np.abs(codebooks[sub]) if sign else codebooks[sub], kind, sub)
    if sign and kind == "inf":
        cb16 = np.abs(cb16)
    cb = torch.from_numpy(cb16).cuda()
    table = api.nsn_build_rope_table(synth.rope_inv_freq(5e5), L) if rope else None
    shape = api.make_shape(sub, H, H, L, 64, sign_format=sign, rope_table=table)
    form = [helpers.encode_launch_form(api, shape, 1, n) for n in (L, PART)]
    assert form[0] == (16, 64, 3) and form[1][0] == 16 and form[1][2] == 2, form
    g = torch.Generator(device="cuda").manual_seed(11)
    k, v = (torch.randn((1, H, L, 128), generator=g, device="cuda").half() for _ in range(2))
    for x in (k, v):
        x[0, 0, 5] = 0.0
        x[0, 1, 70, 1:] = 0.0                       # one channel: equal magnitudes after the rotation
        x[0, 2, 130, 3] = float("nan")              # (in groups of their own: a group's mean takes all of its tokens)
        x[0, 3, 200, 100] = float("inf")
        x[0, 4, 300] *= 1e-3

    def encode(parts):
        caches = api.alloc_cache(shape, 1), api.alloc_cache(shape, 1)
        for at in range(0, L, L // parts):
            n = L // parts
            pos, count = (torch.tensor([x], dtype=torch.int32, device="cuda") for x in (at, n))
            api.nsn_encode(shape, cb, k[:, :, at:at + n].contiguous(), v[:, :, at:at + n].contiguous(), pos, count, *caches)
        torch.cuda.synchronize()
        return caches

    def same(a, b, any_nan=False):  # any_nan: not a number is not a number, whatever its sign (arithmetic leaves that open)
        for x, y in zip(a, b):
            for name in ("codes", "norms", "means"):
                p, q = getattr(x, name), getattr(y, name)
                if any_nan and name != "codes":
                    p, q = (torch.where(t.isnan(), torch.full_like(t, float("nan")), t) for t in (p, q))
                assert torch.equal(p.view(torch.uint8), q.view(torch.uint8)), name

    whole = encode(1)
    same(whole, encode(L // PART))
    assert int((whole[0].codes != 0).sum()) > 0 or kind == "0"
    if not rope and kind not in ("inf", "nan", "nan with its sign set"):
        select_variant("encode", "valu")
        same(whole, encode(1), any_nan=True)
    if kind in ("copies", "edge"):
        later = [r for row, at in (COPIES if kind == "copies" else EDGE) for r in (row, *at) if r != min(row, *at)]
        if not sign:                                # (a sign byte may be any byte)
            assert not np.isin(whole[0].codes.cpu().numpy(), later).any(), "a later copy of a codeword"
