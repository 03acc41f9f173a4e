"""The encoders against the oracle, byte for byte, on inputs where an approximate quotient would go wrong:
numbers on a lattice (half-way points and bin edges are hit exactly), constant and denormal rows, one
large offset under a small spread, and lengths around a page."""
import numpy as np
import pytest
import torch

import paper_2502_00527_amd as pq
from oracle import cache_format, values as ovalues

pytestmark = pytest.mark.gpu
GROUP = 128


def _rows(kind, n, heads, seed):
    """fp16 [n, heads, 128]."""
    rng = np.random.default_rng(seed)
    r = rng.standard_normal((n, heads, 128))
    if kind == "lattice":                       # multiples of a scale: exact half-way points
        r = rng.integers(0, 31, r.shape) * 0.5
    elif kind == "flat":                        # constant rows, and rows whose spread rounds to no scale at all
        r = np.where(rng.random((n, heads, 1)) < 0.5, r[..., :1], 1.0 + 2.0 ** -24 * r)
    elif kind == "denormal":                    # scales below the smallest normal fp16
        r = r * np.exp2(rng.integers(-24, -14, (n, heads, 1)))
    elif kind == "offset":
        r = 1000.0 + 0.5 * r
    elif kind == "wide":                        # differences that are not exact in fp32, sums near the largest fp16
        r = np.clip(r * np.exp2(rng.integers(-24, 15, r.shape)), -65000, 65000)
    return r.astype(np.float16)


@pytest.mark.parametrize("v_bits", [4, 2])
@pytest.mark.parametrize("kind", ["normal", "lattice", "flat", "denormal", "offset", "wide"])
def test_value_encoder_edges(kind, v_bits):
    for n, heads in ((1, 3), (127, 1), (300, 2)):
        v = _rows(kind, n, heads, n)
        codes, s, z = ovalues.quantize_values(v, v_bits)
        want = cache_format.pack_value_page_stream(codes, v_bits, GROUP)
        n_pages = (n + GROUP - 1) // GROUP
        layout = pq.Layout(128, 4, 4, GROUP, heads, 0)
        pool = torch.full((n_pages, pq.pq_vq_bytes_per_page(layout, v_bits)), 0xA5, dtype=torch.uint8, device="cuda:0")
        params = torch.full((n_pages, heads, GROUP, 2), 7.0, dtype=torch.float16, device="cuda:0")
        ids = torch.arange(n_pages, dtype=torch.int32, device="cuda:0")
        pq.pq_encode_values(layout, v_bits, torch.from_numpy(v).to("cuda:0"), ids, pool, params)
        np.testing.assert_array_equal(pool.cpu().numpy().reshape(want.shape), want)
        got = params.permute(0, 2, 1, 3).reshape(n_pages * GROUP, heads, 2).cpu().numpy()
        np.testing.assert_array_equal(got[:n, :, 0].view(np.uint16), s.view(np.uint16))
        np.testing.assert_array_equal(got[:n, :, 1], z)             # (zeros may differ in their sign)
        assert not got[n:].any()
