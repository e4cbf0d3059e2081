"""The means that a call of the encoder forms before it encodes, at the edges of a wave's rounds (16-token steps, 64-token
rounds) and of the chunks: against fp64 sums of the same rounding of the norms.  Rows behind a sequence's tokens hold NaN.
The sums differ from the kernel's in their order only (1e-14), so a stored mean differs by one fp16 step where it lies that close to
the middle of two, and not at all elsewhere."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

COUNTS = [1, 4, 5, 16, 17, 20, 21, 33, 49, 63, 64, 65, 81, 255, 256, 257, 300]


@pytest.mark.parametrize("G", [0, 128, 192])
@pytest.mark.parametrize("sub", [4, 8])
def test_means_at_the_edges(gpu_api, codebooks, sub, G):
    import torch
    api = gpu_api
    B, H, cap = len(COUNTS), 2, 320
    print(f"case sub={sub} G={G}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(8)
    k, v = (torch.randn((B, H, cap, 128), generator=g, device="cuda").half() for _ in range(2))
    k += 3.0
    for b, n in enumerate(COUNTS):
        k[b, :, n:] = float("nan")
        v[b, :, n:] = float("nan")
        v[b, :, n // 2] = 0.0     # a token of zeros adds nothing
    shape = api.make_shape(sub, H, H, 384, G, 0)
    kc, vc = api.alloc_cache(shape, B), api.alloc_cache(shape, B)
    n = torch.tensor(COUNTS, dtype=torch.int32, device="cuda")
    api.nsn_encode(shape, torch.from_numpy(codebooks[sub].astype(np.float16)).cuda(), k, v, torch.zeros_like(n), n, kc, vc)
    torch.cuda.synchronize()
    for c, x in ((kc, k), (vc, v)):
        means, x = c.means.cpu().numpy(), x.double().cpu().numpy()
        for b, count in enumerate(COUNTS):
            s1 = np.sqrt((x[b, :, :count] ** 2).sum(-1, keepdims=True) / 128).astype(np.float16).astype(np.float64)
            y = np.divide(x[b, :, :count], s1, out=np.zeros_like(x[b, :, :count]), where=s1 > 0)
            for i, t in enumerate(range(0, count, G or count)):
                want = y[:, t:t + (G or count)].mean(1)
                got = means[b].reshape(H, -1, 128)[:, i].astype(np.float64)
                # half a step of fp16 above |mean| (of a negative power of two numpy gives the step on its near side)
                half = 0.5 * np.spacing(np.abs(got).astype(np.float16)).astype(np.float64)
                err = np.abs(got - want)
                assert (err <= half * (1 + 1e-6) + 1e-12).all(), (b, count, i, err.max(), got[err > half], want[err > half])
