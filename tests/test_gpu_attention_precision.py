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
