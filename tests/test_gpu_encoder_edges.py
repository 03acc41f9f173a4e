"""The encoders against the oracle, byte for byte, on inputs where an approximate quotient would go wrong:
numbers on a lattice (half-way points and bin edges are hit exactly), constant and denormal rows, one
large offset under a small spread, and lengths around a page."""
import numpy as np
import pytest
import torch

import paper_2502_00527_amd as pq
from oracle import cache_format, polar, values as ovalues

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


@pytest.mark.parametrize("v_bits", [4, 2])
def test_a_nan_stays_where_it_is(v_bits):
    """A NaN among the values has code 0; the other codes, of its own token and of the tokens beside it, and all
    parameters are those of the values without it."""
    n, heads = 300, 2
    for kind in ("normal", "lattice", "denormal", "flat"):
        v = _rows(kind, n, heads, 5)
        rng = np.random.default_rng(6)
        hit = (rng.random(v.shape) < 0.04) & (rng.random((n, heads, 1)) < 0.5)
        hit[7, 0], hit[7, 0, 3] = True, False                       # a token with a single number left
        hit[8] = False
        without = np.where(hit, np.min(np.where(hit, np.float16(np.inf), v), axis=-1, keepdims=True), v)
        with_nan = v.copy()
        with_nan.view(np.uint16)[hit] = rng.choice(np.array([0x7e00, 0xfe00, 0x7fff, 0xffff], np.uint16), int(hit.sum()))
        n_pages = (n + GROUP - 1) // GROUP
        layout = pq.Layout(128, 4, 4, GROUP, heads, 0)
        ids = torch.arange(n_pages, dtype=torch.int32, device="cuda:0")
        got = []
        for values in (with_nan, without):
            pool = torch.full((n_pages, pq.pq_vq_bytes_per_page(layout, v_bits)), 0xA5, dtype=torch.uint8, device="cuda:0")
            params = torch.full((n_pages, heads, GROUP, 2), 7.0, dtype=torch.float16, device="cuda:0")
            pq.pq_encode_values(layout, v_bits, torch.from_numpy(values).to("cuda:0"), ids, pool, params)
            got.append((pool.cpu().numpy(), params.cpu().numpy()))
        np.testing.assert_array_equal(got[0][0], got[1][0], err_msg=kind)
        np.testing.assert_array_equal(got[0][1], got[1][1], err_msg=kind)
        want = cache_format.pack_value_page_stream(ovalues.quantize_values(without, v_bits)[0], v_bits, GROUP)
        np.testing.assert_array_equal(got[0][0].reshape(want.shape), want)


@pytest.mark.parametrize("v_bits", [4, 2])
def test_an_infinity_stays_in_its_row(v_bits):
    """A row with an infinite value has an infinite scale and codes 0; the rows beside it are what they are without it."""
    n, heads = 300, 2
    v = _rows("normal", n, heads, 5)
    hit = np.random.default_rng(6).random((n, heads)) < 0.2
    inf = v.copy()
    inf[hit, 9] = np.inf
    inf[hit & (np.arange(n) % 2 == 0)[:, None], 100] = -np.inf
    n_pages = (n + GROUP - 1) // GROUP
    layout = pq.Layout(128, 4, 4, GROUP, heads, 0)
    pool = torch.full((n_pages, pq.pq_vq_bytes_per_page(layout, v_bits)), 0xA5, dtype=torch.uint8, device="cuda:0")
    params = torch.full((n_pages, heads, GROUP, 2), 7.0, dtype=torch.float16, device="cuda:0")
    ids = torch.arange(n_pages, dtype=torch.int32, device="cuda:0")
    pq.pq_encode_values(layout, v_bits, torch.from_numpy(inf).to("cuda:0"), ids, pool, params)
    codes, s, z = ovalues.quantize_values(v, v_bits)
    want = cache_format.pack_value_page_stream(np.where(hit[..., None], 0, codes), v_bits, GROUP)
    np.testing.assert_array_equal(pool.cpu().numpy().reshape(want.shape), want)
    got = params.permute(0, 2, 1, 3).reshape(n_pages * GROUP, heads, 2).cpu().numpy()[:n]
    assert np.isinf(got[hit][:, 0]).all()
    np.testing.assert_array_equal(got[~hit], np.stack([s, z], axis=-1)[~hit])


def _keys(kind, n, heads, seed, dtype):
    """[n, heads, 128]: keys on which the code's approximation is in doubt, or the quick angle rule does not hold."""
    rng = np.random.default_rng(seed)
    k = rng.standard_normal((n, heads, 128))
    if kind == "lattice":                       # axes, diagonals and the origin; radii that meet bin edges
        k = rng.integers(-15, 16, k.shape) * 0.5
    elif kind == "diagonals":                   # no zeros, |x| = |y| in a quarter of the pairs
        k = rng.choice([-1.0, 1.0], k.shape) * rng.integers(1, 5, k.shape) * 0.25
    elif kind == "zeros":                       # zeros of both signs, a channel without any other number
        k = np.where(rng.random(k.shape) < 0.3, np.copysign(0.0, k), k)
        k[..., 5], k[..., 70] = 0.0, -0.0
    elif kind == "flat":                        # constant radii: scale 0, or a few units of the radius
        k = np.broadcast_to(k[:1], k.shape) * (1 + 2.0 ** -9 * rng.integers(-1, 2, (n, heads, 1)) * (rng.random((1, heads, 1)) < 0.5))
    elif kind == "circle":                      # scales far below the radius
        a = 2 * np.pi * rng.random((n, heads, 64))
        k = 3 * np.concatenate([np.cos(a), np.sin(a)], axis=-1)
    elif kind == "small":                       # fp16 denormals, denormal scales
        k = k * 2.0 ** -20
    elif kind == "wide":
        k = np.clip(k * np.exp2(rng.integers(-24, 12, k.shape)), -20000, 20000)
    return k.astype(dtype)


@pytest.mark.parametrize("rt", [(4, 4), (3, 3), (5, 3), (3, 5), (4, 2), (2, 4)])
@pytest.mark.parametrize("kind", ["normal", "lattice", "diagonals", "zeros", "flat", "circle", "small", "wide"])
def test_key_encoder_edges(kind, rt):
    for n, heads, dtype in ((1, 3, np.float16), (127, 1, np.float32), (300, 2, np.float16), (130, 2, np.float32)):
        k = _keys(kind, n, heads, n, dtype)
        enc = polar.encode_keys(k, *rt, GROUP)
        n_pages = (n + GROUP - 1) // GROUP
        layout = pq.Layout(128, *rt, GROUP, heads, 0)
        codes = torch.full((n_pages, heads, 4, GROUP, 2 * sum(rt)), 0xA5, dtype=torch.uint8, device="cuda:0")
        params = torch.full((n_pages, heads, 64, 2), 7.0, dtype=torch.float16, device="cuda:0")
        order = np.arange(n_pages - 1, -1, -1, dtype=np.int32)                # pages out of order
        pq.pq_encode_keys(layout, torch.from_numpy(k).to("cuda:0"), torch.from_numpy(order).to("cuda:0"), codes, params)
        a, c, s, z = cache_format.unpack_pages(codes.cpu().numpy()[order], params.cpu().numpy()[order], n, *rt)
        np.testing.assert_array_equal(s.view(np.uint16), enc["scale"].view(np.uint16))
        np.testing.assert_array_equal(z.view(np.uint16), enc["zero"].view(np.uint16))
        np.testing.assert_array_equal(c, enc["c"])
        # two float64 evaluations of an irrational edge may differ in the last places
        assert not np.any((a != enc["a"]) & (enc["edge_dist"] > 1e-12))
        assert not codes.cpu().numpy()[order][-1, :, :, n - (n_pages - 1) * GROUP:].any()


@pytest.mark.parametrize("n", [1, 8, 9, 33, 64, 97, 127, 129])
def test_grouped_angles_of_partial_pages(n):
    """Whole steps of a wavefront lie past the end: they have no say in the group's angles."""
    for dtype, rt in ((np.float16, (4, 4)), (np.float32, (3, 5))):
        k = _keys("normal", n, 2, n, dtype)
        enc = polar.encode_keys(k, *rt, GROUP, grouped_angles=True)
        n_pages = (n + GROUP - 1) // GROUP
        layout = pq.Layout(128, *rt, GROUP, 2, 1)
        codes = torch.full((n_pages, 2, 4, GROUP, 2 * sum(rt)), 0xA5, dtype=torch.uint8, device="cuda:0")
        params = torch.full((n_pages, 2, 2, 64, 2), 7.0, dtype=torch.float16, device="cuda:0")
        pq.pq_encode_keys(layout, torch.from_numpy(k).to("cuda:0"), torch.arange(n_pages, dtype=torch.int32, device="cuda:0"), codes, params)
        a, c, s, z, ts, tz = cache_format.unpack_pages(codes.cpu().numpy(), params.cpu().numpy(), n, *rt)
        for got, want in ((s, "scale"), (z, "zero"), (ts, "t_scale"), (tz, "t_zero")):
            np.testing.assert_array_equal(got.view(np.uint16), enc[want].view(np.uint16))
        np.testing.assert_array_equal(c, enc["c"])
        assert not np.any((a != enc["a"]) & (enc["edge_dist"] > 1e-12))


def test_more_work_groups_than_one_launch_takes():
    """2^24 work-groups of 256 threads are more than a grid may have: the encoders launch in parts.  The heads are views of
    one row, and only pages before, across and behind the parts' border have a place in the pools."""
    heads, groups = 4096, 4200
    part = (2 ** 24 - 1) // heads
    n = groups * GROUP - 5
    g = torch.Generator(device="cuda:0")
    g.manual_seed(1)
    rows = torch.randn((n, 1, 128), generator=g, device="cuda:0", dtype=torch.float16)
    kept = [3, part - 1, part, groups - 1]
    ids = torch.full((groups,), -1, dtype=torch.int32)
    ids[kept] = torch.arange(4, dtype=torch.int32)
    ids = ids.to("cuda:0")
    pools = []
    for h in (heads, 1):
        layout = pq.Layout(128, 3, 3, GROUP, h, 0)
        codes = torch.zeros((4, h, 4 * GROUP * 12), dtype=torch.uint8, device="cuda:0")
        params = torch.zeros((4, h, 64, 2), dtype=torch.float16, device="cuda:0")
        vq = torch.zeros((4, h, GROUP * 128 // 4), dtype=torch.uint8, device="cuda:0")
        vq_params = torch.zeros((4, h, GROUP, 2), dtype=torch.float16, device="cuda:0")
        if h > 1:
            pq.pq_encode_keys(layout, rows.expand(n, h, 128), ids, codes, params)
            pq.pq_encode_values(layout, 2, rows.expand(n, h, 128), ids, vq, vq_params)
        else:
            for page, group in enumerate(kept):
                at = torch.tensor([page], dtype=torch.int32, device="cuda:0")
                pq.pq_encode_keys(layout, rows[group * GROUP:(group + 1) * GROUP], at, codes, params)
                pq.pq_encode_values(layout, 2, rows[group * GROUP:(group + 1) * GROUP], at, vq, vq_params)
        pools.append((codes, params, vq, vq_params))
    for many, one in zip(*pools):
        assert torch.equal(many, one.expand_as(many)) and bool(one.any())
