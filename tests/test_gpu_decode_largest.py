"""The largest cache a shape may have: sequences that end at or just below token 2^31 - 64, where sums of token indices leave 31
bits.  Only the last tokens count (all others score more than 80 nats less), so the result is that of a short cache that holds
those alone; rounding differs by the weights' fp16 factor (relative 2^-11 each, as between any two split counts)."""
import math

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

MAX_LEN, TAIL = (1 << 31) - 64, 4096 + 64
PAGE = MAX_LEN // 1801


@pytest.fixture(scope="module")
def buffers():
    """Codes and norms of every test here, K and V alike (40 GiB)."""
    codes = torch.zeros(MAX_LEN * 16, dtype=torch.uint8, device="cuda")
    norms = torch.zeros(MAX_LEN * 2, dtype=torch.float16, device="cuda")
    yield codes, norms
    del codes, norms
    torch.cuda.empty_cache()


@pytest.mark.parametrize("impl,n_splits,side_bits,page,short", [
    ("mfma", 64, 16, 0, 17), ("mfma", 0, 16, 0, 0), ("mfma", 64, 4, 0, 0), ("mfma", 0, 4, 0, 17),
    ("mfma", 64, 16, PAGE, 17), ("mfma", 0, 16, PAGE, 0), ("lut", 64, 16, 0, 17)])
def test_sequences_that_end_below_2_31(gpu_api, select_variant, buffers, impl, n_splits, side_bits, page, short):
    api = gpu_api
    print(f"case {impl} splits={n_splits} side_bits={side_bits} page={page} short={short}", flush=True)
    select_variant("decode", impl)
    g = torch.Generator(device="cuda").manual_seed(5)
    codes, norms = buffers
    cb = torch.randn((256, 8), generator=g, device="cuda").half()
    q = torch.randn((1, 1, 128), generator=g, device="cuda").abs().add(0.5).half()
    k_mean = torch.full((128,), -8.0, device="cuda").half()      # q . o^k / sqrt(d) is -90 or less: a token with b = 1 does not count
    v_mean = torch.randn((128,), generator=g, device="cuda").half()
    tail_codes = torch.randint(0, 256, (TAIL * 16,), generator=g, device="cuda", dtype=torch.uint8)
    rand = lambda lo, hi, *n: torch.rand(n, generator=g, device="cuda").mul(hi - lo).add(lo).half()
    if side_bits == 16:
        record = torch.tensor([0.0, 1.0], device="cuda").half().view(torch.uint8).view(1, 4)        # (a, b)
        tail_norms = torch.stack([rand(0.5, 1.5, TAIL), rand(0.0, 0.02, TAIL)], dim=1).view(torch.uint8)
    else:  # 64 a', 64 four-bit codes of b, (min, step) of b
        record = torch.zeros((1, 164), dtype=torch.uint8, device="cuda")
        record[0, 160:162] = torch.tensor([1.0], device="cuda").half().view(torch.uint8)
        tail_norms = torch.cat([rand(25.0, 75.0, TAIL // 64, 64).view(torch.uint8),
                                torch.randint(0, 256, (TAIL // 64, 32), generator=g, device="cuda", dtype=torch.uint8),
                                torch.tensor([[0.005, 0.001]], device="cuda").half().view(torch.uint8).expand(TAIL // 64, 4)], dim=1)
    rows = MAX_LEN if side_bits == 16 else MAX_LEN // 64
    far_norms = norms.view(torch.uint8)[:rows * record.shape[1]].view(rows, record.shape[1])
    far_norms.copy_(record.expand(rows, -1))

    def caches(shape, c, n, table):
        out = []
        for mean in (k_mean, v_mean):
            if side_bits == 16:
                m = mean.view(1, 1, 1, 128).clone()
            else:  # 64 bytes of codes, four (min, step): the first is the value of a group's channels, or 1/8 steps of code 1..15
                m = torch.zeros((1, 1, 1, 80), dtype=torch.uint8, device="cuda")
                par = torch.tensor([[-8.0, 0.0] if mean is k_mean else [-1.0, 0.125]] * 4, device="cuda").half()
                m[..., 64:] = par.view(torch.uint8).flatten()
                if mean is v_mean:
                    m[..., :64] = torch.arange(64, dtype=torch.uint8, device="cuda") * 37
            out.append(api.CodedCache(c, n, m, table))
        return out

    table = None
    end = MAX_LEN
    if page:  # the sequence's last page is the buffer's first
        table = torch.arange(1800, -1, -1, dtype=torch.int32, device="cuda").view(1, 1801)
        end = page
    per_row = MAX_LEN // rows
    codes[(end - TAIL) * 16:end * 16] = tail_codes
    far_norms[(end - TAIL) // per_row:end // per_row] = tail_norms
    big = api.make_shape(8, 1, 1, MAX_LEN, 0, page, side_bits=side_bits)
    small = api.make_shape(8, 1, 1, TAIL, 0, side_bits=side_bits)
    assert api.nsn_max_groups(big) == 1
    scale = 1.0 / math.sqrt(128)

    def attend(shape, kv, n, splits):
        lens = torch.tensor([n], dtype=torch.int32, device="cuda")
        return api.nsn_decode_attention(shape, cb, q, *kv, lens, n, scale, n_splits=splits)

    ref = attend(small, caches(small, tail_codes, tail_norms, None), TAIL - short, 1)
    torch.cuda.synchronize()
    out = attend(big, caches(big, codes, far_norms, table), MAX_LEN - short, n_splits)
    torch.cuda.synchronize()
    codes[(end - TAIL) * 16:end * 16] = 0
    err = float((out - ref).abs().max() / ref.abs().max())
    print(f"  max rel err {err:.2e}", flush=True)
    assert err < 2e-3, err
