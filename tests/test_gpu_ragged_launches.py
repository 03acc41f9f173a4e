"""Launches whose chunks are cut by the sequences' real lengths (at least 48 * 512 pages times KV heads if
every sequence had max_seq_len tokens): max_seq_len far above the lengths, one long sequence among
short ones, empty ones, more sequences than a wavefront has lanes, several passes over the query
heads, and the same with the raw scores asked for.  Against float64."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _lens(kind):
    """Lengths, all far below the launch's max_seq_len."""
    rng = np.random.default_rng(3)
    if kind == "loose":
        return [260] * 16
    if kind == "one_long":                                             # 40 pages and 31 x 1: several chunks of one sequence
        return [5100] + [100] * 31
    if kind == "long_in_the_middle":
        return [130] * 20 + [9000] + [0] * 3 + [700] * 9
    if kind == "ragged":
        return [int(x) for x in rng.integers(1, 2600, 40)]
    if kind == "seventy":                                              # a second block of sequences, the long one in it
        return [int(x) for x in rng.integers(0, 300, 68)] + [3900, 1]
    if kind == "all_empty_but_one":
        return [0] * 63 + [1]
    if kind == "five_hundred_and_twelve":
        return [int(x) for x in rng.integers(1, 140, 511)] + [1500]
    raise ValueError(kind)


CASES = [(kind, group, v_bits, scores) for kind in ("loose", "one_long", "long_in_the_middle", "ragged", "seventy", "all_empty_but_one",
                                                   "five_hundred_and_twelve")
         for group, v_bits, scores in ((4, 16, False), (1, 4, False), (7, 2, True), (12, 16, True))]


@pytest.mark.parametrize("kind,group,v_bits,scores", CASES)
def test_lengths_below_the_bound(kind, group, v_bits, scores):
    from packed import Packed, relative_error

    import paper_2502_00527_amd as pq

    lens = _lens(kind)
    heads = 1 if len(lens) > 100 else 4
    max_seq_len = max(max(lens), (48 * 512 + len(lens) * heads - 1) // (len(lens) * heads) * 128)
    rng = np.random.default_rng(len(lens))
    keys = [rng.standard_normal((n, heads, 128)).astype(np.float16) for n in lens]
    values = [rng.standard_normal((n, heads, 128)).astype(np.float32) for n in lens]
    q = rng.standard_normal((len(lens), heads * group, 128)).astype(np.float16)
    cache = Packed(keys, values, q, v_bits=v_bits, max_seq_len=max_seq_len)
    assert pq.pq_decode_merges_in_kernel(cache.layout, len(lens), heads * group, max_seq_len, v_bits)
    raw = torch.full((len(lens), heads * group, max_seq_len), float("nan"), device="cuda:0") if scores else None
    out = cache.attention(raw)
    want_scores, want = cache.exact()
    for s, n in enumerate(lens):
        if n == 0:
            assert not bool(out[s].any()), "an empty sequence gives zero rows"
            want[s] = 0.0
    err = relative_error(out, want)
    print(f"[ragged] {kind} group {group} v{v_bits}: {err:.2e}", flush=True)
    assert err <= (2e-6 if v_bits == 16 else 2.4e-5)
    assert torch.equal(out, cache.attention(raw))
    if scores:
        for s, n in enumerate(lens):
            assert bool(torch.isnan(raw[s, :, n:]).all())
        got_scores = torch.cat([raw[s, :, :n].cpu().reshape(-1) for s, n in enumerate(lens)])
        # 9.2e-8 over many scores, to a few per cent; a single token's 28 scatter (each is rounded 19 times on the
        # way, 19 * 2^-25 at most of its partial sums' size)
        assert relative_error(got_scores, torch.cat([w.reshape(-1) for w in want_scores])) <= (1.05e-7 if sum(lens) > 100 else 19 * 2.0 ** -25)
