"""Attention against float64 where 16-bit parts of a number would show: softmaxes that hang on few
tokens, values and parameters far from 1.

Bounds.  A score carries 1e-7 of its size (22-bit factors, fp32 sums), an exponential twice that; a
softmax of logits up to 17 is therefore good to 17 * 1e-7 + 2^-22, 2e-6, as fp32 arithmetic is.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _random(seed, *shape):
    return np.random.default_rng(seed).standard_normal(shape).astype(np.float32)


@pytest.mark.parametrize("v_bits", [16])
@pytest.mark.parametrize("group", [1, 4, 8])
@pytest.mark.parametrize("logit", [8.0, 11.0, 14.0, 17.0])
def test_attention_sinks(group, logit, v_bits):
    """One token in every page takes nearly all the weight and has a zero value row, so that the output is
    made of the weights of the others: 2^-11 to 2^-25 of the largest."""
    from packed import Packed, relative_error

    heads, length = 2, 1500
    keys, values = _random(1, length, heads, 128), _random(2, length, heads, 128)
    direction = _random(3, heads, 128)
    direction /= np.linalg.norm(direction, axis=-1, keepdims=True)
    keys[::128] = np.sqrt(128.0) * direction
    values[::128] = 0.0
    q = _random(4, 1, heads, group, 128) + logit * direction[:, None]
    cache = Packed([keys.astype(np.float16)], [values], q.reshape(1, -1, 128).astype(np.float16), v_bits=v_bits)
    _, want = cache.exact()
    err = relative_error(cache.attention(), want)
    print(f"[precision] sinks group {group} logit {logit} v{v_bits}: {err:.2e}", flush=True)
    assert err <= 4e-6


@pytest.mark.parametrize("v_bits", [16, 4, 2])
@pytest.mark.parametrize("exponent", [8, -4, -7, -10])
@pytest.mark.parametrize("sharpness", [0.4, 1.0, 3.0])
def test_values_of_any_size(sharpness, exponent, v_bits):
    """Values times a power of two give outputs times it: scales of 2^-10 are no harder than scales of 1.
    With quantized values out = sum p (code s) + sum p z cancels (|z| is up to 100 times a flat softmax's
    output), and fp32 sums of both parts leave up to 100 * 2^-22."""
    from packed import Packed, relative_error

    heads, length, group = 2, 3000, 4
    keys, values = _random(5, length, heads, 128), _random(6, length, heads, 128) * 2.0 ** exponent
    q = _random(7, 1, heads * group, 128) * sharpness
    cache = Packed([keys.astype(np.float16)], [values], q.astype(np.float16), v_bits=v_bits)
    err = relative_error(cache.attention(), cache.exact()[1])
    print(f"[precision] values 2^{exponent} sharpness {sharpness} v{v_bits}: {err:.2e}", flush=True)
    assert err <= (2e-6 if v_bits == 16 else 2.4e-5)


@pytest.mark.parametrize("v_bits", [16, 4, 2])
@pytest.mark.parametrize("order", [1, -1])
def test_values_of_all_sizes_at_once(order, v_bits):
    """Sizes of 2^-12 to 2^10 from page to page, growing and shrinking along the context, with the weights
    on the small ones; two tokens of a page differ by 2^8."""
    from packed import Packed, relative_error

    heads, length, group = 2, 2900, 4
    keys, values = _random(8, length, heads, 128), _random(9, length, heads, 128)
    size = np.linspace(-12, 10, length)[::order][:, None, None]
    values *= np.exp2(np.round(size)) * np.where(np.arange(length) % 2, 1.0, 2.0 ** -8)[:, None, None]
    direction = _random(10, heads, 128)
    direction /= np.linalg.norm(direction, axis=-1, keepdims=True)
    keys -= direction * size * np.log(2.0) * 2.0                                    # weight ~ 1 / size
    q = _random(11, 1, heads, group, 128) * 0.3 + direction[:, None] * np.sqrt(128.0) * 0.5
    cache = Packed([keys.astype(np.float16)], [values], q.reshape(1, -1, 128).astype(np.float16), v_bits=v_bits)
    err = relative_error(cache.attention(), cache.exact()[1])
    print(f"[precision] values of all sizes order {order} v{v_bits}: {err:.2e}", flush=True)
    assert err <= (4e-6 if v_bits == 16 else 2.4e-5)


@pytest.mark.parametrize("group", [1, 4, 8])
def test_infinite_value_elements(group):
    """A value element that is infinite makes that element of the output infinite, and no other."""
    from packed import Packed

    heads, length = 2, 700
    keys, values = _random(12, length, heads, 128), _random(13, length, heads, 128)
    values[3, 0, 5], values[200, 0, 17], values[650, 1, 40] = np.inf, -np.inf, np.inf
    cache = Packed([keys.astype(np.float16)], [values], _random(14, 1, heads * group, 128).astype(np.float16))
    got, want = cache.attention().cpu().double(), cache.exact()[1]
    assert int(torch.isinf(want).sum()) == 3 * group
    assert torch.equal(torch.isinf(got), torch.isinf(want)) and torch.equal(got[torch.isinf(want)], want[torch.isinf(want)])
    assert float((got - want)[torch.isfinite(want)].abs().max()) <= 1e-5


@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("group", [1, 4, 5, 8])
@pytest.mark.parametrize("radius", [1.0, 400.0, 30000.0])
def test_raw_scores_carry_fp32(radius, group, dtype):
    """Raw scores are fp32 multiply-adds, whatever the query group, and whatever the size of one pair's
    radius beside the others' (the query is zero there): 9.2e-8 of the scores' 2-norm; the same through
    pq_decode_attention."""
    from packed import Packed, relative_error

    heads, length = 2, 1300
    keys = _random(15, length, heads, 128)
    keys[..., 5], keys[..., 69] = radius, 0.0
    q = _random(16, 1, heads * group, 128)
    q[..., 5] = q[..., 69] = 0.0
    cache = Packed([keys.astype(dtype)], [_random(17, length, heads, 128)], q.astype(dtype))
    want = cache.exact()[0][0]
    got = cache.scores()
    err = relative_error(got[0], want)
    print(f"[precision] scores radius {radius} group {group} {dtype.__name__}: {err:.2e}", flush=True)
    assert err <= 1.05e-7
    through_attention = torch.full_like(got, float("nan"))
    cache.attention(through_attention)
    assert torch.equal(through_attention, got)


@pytest.mark.parametrize("group", [2, 8])
def test_score_rows_a_gibibyte_apart(group):
    """pq_decode_attention takes any scores_stride; rows further apart than 32-bit offsets of 4 rows reach
    are written one at a time."""
    from packed import Packed

    length = 300
    cache = Packed([_random(18, length, 1, 128).astype(np.float16)], [_random(19, length, 1, 128)],
                   _random(20, 1, group, 128).astype(np.float16))
    near = torch.full((1, group, length), float("nan"), device="cuda:0")
    want = cache.attention(near)
    far = torch.full((1, group, (1 << 28) + 3), float("nan"), device="cuda:0")
    assert torch.equal(cache.attention(far), want)
    assert torch.equal(far[..., :length], near)
    assert bool(torch.isnan(far[..., length:]).all())


@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("group", [1, 4, 8])
@pytest.mark.parametrize("radius", [16.0, 400.0, 30000.0])
@pytest.mark.parametrize("tail", [0, 50])
@pytest.mark.parametrize("zero_heads", [0, 1, 2])
def test_one_large_radius(zero_heads, tail, radius, group, dtype):
    """Keys whose pair 5 is far larger than the others, with queries that are small there by as much, or
    zero -- for no head, every second one or all: the other pairs decide the softmax.  With a tail of
    un-quantized keys too."""
    from packed import Packed, relative_error

    heads, length = 2, 1280 + tail
    keys = _random(21, length, heads, 128) * 0.25
    keys[..., 5], keys[..., 69] = radius, 0.0
    q = _random(22, 1, heads * group, 128)
    q[..., 5] /= radius
    q[..., 69] /= radius
    if zero_heads:
        q[:, ::3 - zero_heads, 5] = q[:, ::3 - zero_heads, 69] = 0.0
    cache = Packed([keys.astype(dtype)], [_random(23, length, heads, 128)], q.astype(dtype), residual=tail > 0)
    err = relative_error(cache.attention(), cache.exact()[1])
    print(f"[precision] radius {radius} zero {zero_heads} group {group} {dtype.__name__} tail {tail}: {err:.2e}", flush=True)
    assert err <= 1e-6


@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("group", [1, 4, 8])
@pytest.mark.parametrize("size", [1000.0, 30000.0])
def test_one_large_query_element(size, group, dtype):
    """The other way round: the query's largest element meets keys that are small there."""
    from packed import Packed, relative_error

    heads, length = 2, 1400
    keys = _random(24, length, heads, 128)
    keys[..., 7], keys[..., 71] = 1.0 / size, 0.5 / size
    q = _random(25, 1, heads * group, 128)
    q[..., 7] = size
    cache = Packed([keys.astype(dtype)], [_random(26, length, heads, 128)], q.astype(dtype))
    err = relative_error(cache.attention(), cache.exact()[1])
    print(f"[precision] query element {size} group {group} {dtype.__name__}: {err:.2e}", flush=True)
    assert err <= 1e-6
