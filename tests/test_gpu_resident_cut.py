"""Launches whose sequences leave places on the compute units: their chunks are cut on the device so that all start at once, and
dealt out by length (or as the host cut them, if the sequences are as long as it was told; or by the general rule, if too
many are left).  Every chunk has to be somebody's, whatever the lengths: more and fewer sequences than compute units per KV
head, KV heads that do not divide 256, units without a first chunk, empty sequences, chunks of equal and of very different
lengths, a bound far above the lengths.  Against float64; the same bits on a second call."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _case(kind):
    """KV heads, lengths, max_seq_len (pages times KV heads if every sequence had it: above 4 * 512, two chunks or more)."""
    rng = np.random.default_rng(11)
    if kind == "alike":                                                # as long as the bound: the host's chunks
        return 8, [16 * 128] * 17, 16 * 128
    if kind == "alike_below_the_bound":
        return 4, [700] * 20, 6000
    if kind == "spread":
        return 4, [int(x) for x in rng.integers(1, 3400, 20)], 3400
    if kind == "more_than_units":                                      # 40 sequences on 32 units a KV head
        return 8, [int(x) for x in rng.integers(1, 1300, 40)], 1500
    if kind == "one_long":                                             # most units have nothing but a first chunk of one page
        return 2, [6000] + [1 + i for i in range(40)], 6000
    if kind == "three_heads":
        return 3, [int(x) for x in rng.integers(1, 4000, 23)], 5000
    if kind == "seven_heads":
        return 7, [0, 2900, 5, 0, 128, 129, 1000, 2432, 2433], 4500
    if kind == "two_sequences":                                        # units without a first chunk take the longest others
        return 16, [2300, 400], 9000
    if kind == "sixty_four":
        return 2, [int(x) for x in rng.integers(0, 800, 63)] + [2100], 2500
    if kind == "too_many":                                             # no cut fits: the general rule
        return 8, [1664] * 33, 1920
    if kind == "large":                                                # 48 * 512 pages by the bound
        return 4, [int(x) for x in rng.integers(1, 2500, 6)], 6 * 196608 // 4
    raise ValueError(kind)


KINDS = ["alike", "alike_below_the_bound", "spread", "more_than_units", "one_long", "three_heads", "seven_heads", "two_sequences",
         "sixty_four", "too_many", "large"]
CASES = [(kind, group, v_bits, rt) for i, kind in enumerate(KINDS)
         for group, v_bits, rt in (((1, 16, (4, 4)), (6, 2, (3, 3))) if i % 2 else ((4, 4, (4, 4)), (2, 16, (3, 3))))
         if kind != "too_many" or group == 1]


@pytest.mark.parametrize("kind,group,v_bits,rt", CASES)
def test_every_chunk_is_taken(kind, group, v_bits, rt):
    from packed import Packed, relative_error

    import paper_2502_00527_amd as pq

    heads, lens, max_seq_len = _case(kind)
    rng = np.random.default_rng(len(lens))
    keys = [rng.standard_normal((n, heads, 128)).astype(np.float16) for n in lens]
    values = [rng.standard_normal((n, heads, 128)).astype(np.float32) for n in lens]
    q = rng.standard_normal((len(lens), heads * group, 128)).astype(np.float16)
    cache = Packed(keys, values, q, v_bits=v_bits, max_seq_len=max_seq_len, bits=rt)
    assert pq.pq_decode_merges_in_kernel(cache.layout, len(lens), heads * group, max_seq_len, v_bits)
    out = cache.attention()
    want = cache.exact()[1]
    for s, n in enumerate(lens):
        if n == 0:
            assert not bool(out[s].any()), "an empty sequence gives zero rows"
            want[s] = 0.0
        # sequence by sequence: a chunk that nobody took would show in its own row
        err = relative_error(out[s], want[s]) if n else 0.0
        assert err <= (4e-6 if v_bits == 16 else 1e-4), (s, n, err)
    err = relative_error(out, want)
    print(f"[resident cut] {kind} group {group} v{v_bits}: {err:.2e}", flush=True)
    assert err <= (2e-6 if v_bits == 16 else 2.4e-5)
    assert torch.equal(out, cache.attention())


# sequences, KV heads, longest and shortest context
GROUPED = [(20, 8, 2000, 1), (9, 16, 2050, 300), (40, 4, 1800, 1), (17, 8, 2048, 2048)]


@pytest.mark.parametrize("bits", [(4, 4), (3, 3), (5, 3), (3, 5), (4, 2), (2, 4)])
@pytest.mark.parametrize("v_bits,group,dtype", [(16, 3, "f16"), (16, 7, "f32"), (4, 4, "f32"), (4, 12, "f16"), (2, 4, "f16"), (2, 8, "f16")])
def test_grouped_quantizer(bits, v_bits, group, dtype):
    """The same cut with the grouped angle quantizer (three query heads per KV head and more); bounds as in test_gpu_grouped_matrix.py."""
    from perf import cases

    import paper_2502_00527_amd as pq

    seqs, heads, longest, shortest = GROUPED[(sum(bits) + bits[0] + v_bits + group) % len(GROUPED)]
    case = cases._case("cut", "decode", seqs, heads * group, heads, longest, min_context=shortest, r_bits=bits[0], t_bits=bits[1], v_bits=v_bits,
                       dtype=dtype, shuffled_pages=True, grouped_angles=True)
    print("[resident cut]", case, flush=True)
    state = cases.prepare(case, 3)
    assert pq.pq_decode_merges_in_kernel(state["layout"], seqs, heads * group, state["max_seq_len"], v_bits)
    got, want = cases.run(state).clone(), cases.exact(case, 3)
    for s in range(seqs):
        err = float((got[s].double() - want[s]).norm() / want[s].norm())
        assert err <= (1.2e-5 if v_bits == 16 else 1e-4), (s, err)
    err = float((got.double() - want).norm() / want.norm())
    assert err <= (6e-6 if v_bits == 16 else 4e-5), err
    assert torch.equal(got, cases.run(state))
