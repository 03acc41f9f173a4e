"""The attention kernel's dispatch edges (chunk plans, heads per pass, query types) and the value
quantizer's near-half rule, on inputs made for them.

Attention is compared with float64 attention over the same packed cache (perf/cases.py builds both
with plain torch).  Bounds: scores carry 22-bit factors and fp32 sums, exponentials 2^-23 -- 3e-6 of the
output's 2-norm, as the fp16-value cases state; with quantized values out = sum p (code s) + sum p z
cancels (|z| is 60 - 100 times the output's size for flat softmaxes), and fp32 sums of both parts
leave up to 100 * 2^-22 = 2.4e-5; 4e-5 here.
"""
import pytest

torch = pytest.importorskip("torch")

# name, sequences, query heads, KV heads, longest and shortest context, value bits, query type
PLANS = [
    ("one_chunk", 1, 32, 8, 895, 895, 16, "f16"),               # 7 pages: a single chunk, written directly
    ("merge_kernel_two_chunks", 2, 32, 8, 1024, 1000, 16, "f16"),   # 8 pages, few units: partials and merge kernel
    ("sixteen_page_chunks", 31, 32, 8, 3001, 129, 16, "f32"),   # merged in the kernel, odd number of sequences
    ("big_chunks", 8, 32, 8, 32768, 1, 16, "f16"),              # equal big chunks, fp16 values
    ("big_then_small", 70, 8, 8, 8321, 1, 16, "f16"),           # more than 64 pages a share: two chunk lengths, cut on the device
    ("quantized_big_then_small", 20, 32, 8, 8192, 1, 4, "f16"),
    ("quantized_2bit_tail", 40, 14, 2, 8449, 100, 2, "f32"),    # 7 heads in one pass
    ("five_heads", 3, 40, 8, 1500, 7, 16, "f32"),
    ("sixteen_heads", 3, 32, 2, 2049, 2048, 16, "f16"),         # two passes of 8
]


# one launch does everything, or the merge kernel follows
SEPARATE_MERGE = {"merge_kernel_two_chunks", "five_heads", "sixteen_heads"}

# every allocation on the small shapes; the others differ in the key-side table only
CASES = [(p, b) for p in PLANS for b in [(4, 4), (3, 3), (3, 5), (2, 4), (5, 3), (4, 2)] if p[1] <= 8 or b in ((4, 4), (3, 3))]


@pytest.mark.gpu
@pytest.mark.parametrize("plan,bits", CASES, ids=lambda x: x[0] if isinstance(x[0], str) else f"r{x[0]}t{x[1]}")
def test_attention_against_float64(plan, bits):
    import paper_2502_00527_amd as pq
    from perf import cases

    name, seqs, q_heads, kv_heads, context, shortest, v_bits, dtype = plan
    case = cases._case(name, "decode", seqs, q_heads, kv_heads, context, min_context=shortest, v_bits=v_bits,
                       dtype=dtype, r_bits=bits[0], t_bits=bits[1], shuffled_pages=True)
    print(f"[matrix] {name} {bits}", flush=True)
    state = cases.prepare(case, 5)
    merges = pq.pq_decode_merges_in_kernel(state["layout"], seqs, q_heads, state["max_seq_len"], v_bits)
    assert merges == (name not in SEPARATE_MERGE), "the case no longer reaches the plan it is named after"
    state["workspace"].fill_(0x5A)                              # arrival words need no initialisation
    first = cases.run(state).clone()
    second = cases.run(state)
    torch.cuda.synchronize()
    assert torch.equal(first, second)                           # chunks are combined in chunk order
    want = cases.exact(case, 5)
    err = float((first.double() - want).norm() / want.norm())
    assert err <= (3e-6 if v_bits == 16 else 4e-5), err


@pytest.mark.gpu
def test_negative_and_zero_softmax_scale():
    """The scale's sign goes into the query; a zero scale gives the mean of the values."""
    from perf import cases

    case = cases._case("scale", "decode", 2, 8, 2, 700, min_context=300)
    state = cases.prepare(case, 3)
    plus = cases.run(state).clone()
    state["q"] = -state["q"]
    state["sm_scale"] = -state["sm_scale"]
    assert torch.equal(cases.run(state), plus)
    state["sm_scale"] = 0.0
    out = cases.run(state).double().view(2, 2, 4, 128)
    for s, n in enumerate(cases._lengths(case)):
        mean = cases._values(case, 3, s, n).double().mean(dim=0)                       # [KV heads, d]
        assert float((out[s] - mean[:, None]).abs().max()) <= 1e-5


@pytest.mark.gpu
@pytest.mark.parametrize("v_bits", [4, 2])
def test_value_codes_at_halves(v_bits):
    """Quotients on and next to k + 1/2, where the product with 1 / s may not decide."""
    import numpy as np

    import paper_2502_00527_amd as pq
    from oracle import cache_format, values as ovalues

    levels = 2 ** v_bits - 1
    rows = []
    for scale in (1.0, 0.25, 3.0, 0.1, 7.0e-5, 1000.0):
        for zero in (0.0, -2.0, 0.37):
            s, z = np.float16(scale), np.float16(zero)
            at = z + (np.arange(128) % (2 * levels + 1) / 2).astype(np.float32) * np.float32(s)
            row = at.astype(np.float16)
            row[0], row[1] = z, np.float16(np.float32(z) + levels * np.float32(s))
            rows += [row, np.nextafter(row, np.float16(np.inf)), np.nextafter(row, np.float16(-np.inf))]
    v = np.stack(rows + [np.zeros(128, np.float16), np.full(128, 5, np.float16)])[:, None]      # [L, 1, 128]
    layout = pq.Layout(128, 4, 4, 128, 1)
    pool = torch.zeros((1, 1, 128 * v_bits // 16, 16, 16), dtype=torch.uint8, device="cuda:0")
    params = torch.zeros((1, 1, 128, 2), dtype=torch.float16, device="cuda:0")
    pq.pq_encode_values(layout, v_bits, torch.from_numpy(v).cuda(), torch.zeros(1, dtype=torch.int32, device="cuda:0"),
                        pool, params)
    torch.cuda.synchronize()
    codes, s, z = ovalues.quantize_values(v, v_bits)
    np.testing.assert_array_equal(pool.cpu().numpy().ravel(), cache_format.pack_value_page_stream(codes, v_bits, 128).ravel())
    got = params.cpu().numpy().view(np.uint16)[0, 0, : len(v)]
    np.testing.assert_array_equal(got, np.stack([s[:, 0], z[:, 0]], axis=-1).view(np.uint16))
