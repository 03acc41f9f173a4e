"""The grouped angle quantizer's kernels on the matrix cores (3 to 16 query heads per KV head): passes of 3 to 8 heads, every
allocation and value width, edges of pages and chunks, un-quantized tails, raw scores, and inputs of very different sizes.

Against float64 over the same packed cache (perf/cases.py builds both with plain torch).  The hardware's sine and
cosine are good to about 2^-21 of a unit and enter the scores of 64 pairs; fp32 arithmetic has 4e-7 - 9e-7 of the
output's norm on such inputs, 3.5e-6 where a single key dominates: 6e-6 is the bound, 4e-5 with quantized values (as in
test_gpu_matrix_attention.py)."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# op, sequences, query heads, KV heads, longest and shortest context, value bits, query type
SHAPES = [
    ("decode", 2, 24, 8, 1000, 1000, 16, "f16"), ("decode", 3, 8, 2, 129, 1, 16, "f32"), ("decode", 1, 5, 1, 5000, 5000, 16, "f16"),
    ("decode", 5, 14, 2, 700, 100, 4, "f32"), ("decode", 2, 16, 2, 1281, 1280, 2, "f16"), ("decode", 40, 32, 4, 640, 1, 16, "f16"),
    ("decode", 2, 24, 2, 900, 20, 4, "f16"), ("serve", 7, 32, 8, 700, 20, 16, "f16"), ("serve", 5, 16, 1, 300, 100, 2, "f32"),
    ("score", 3, 12, 4, 1000, 3, 16, "f16"), ("score", 2, 32, 2, 2049, 127, 16, "f16"), ("score", 2, 8, 1, 515, 515, 16, "f32"),
]


@pytest.mark.parametrize("bits", [(4, 4), (3, 3), (5, 3), (3, 5), (4, 2), (2, 4)])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_against_float64(shape, bits):
    from perf import cases

    op, seqs, q_heads, kv_heads, context, shortest, v_bits, dtype = shape
    case = cases._case("grouped", op, seqs, q_heads, kv_heads, context, min_context=shortest, v_bits=v_bits, dtype=dtype,
                       r_bits=bits[0], t_bits=bits[1], shuffled_pages=True, grouped_angles=True)
    print("[grouped]", shape, bits, flush=True)
    state = cases.prepare(case, 5)
    if op == "score":
        state["scores"].fill_(0.0)
    got, want = cases.run(state), cases.exact(case, 5)
    if op == "serve":
        got, want = got[0], want[0]
    err = float((got.double() - want).norm() / want.norm())
    assert err <= (5e-7 if op == "score" else 6e-6 if v_bits == 16 else 4e-5), err


@pytest.mark.parametrize("q_heads", [3, 4, 6, 8, 12])
@pytest.mark.parametrize("dtype", ["f16", "f32"])
def test_output_does_not_depend_on_the_scores(q_heads, dtype):
    """`out` is the same bit for bit whether raw scores are asked for; they are those of pq_score_keys."""
    from perf import cases

    pq = cases.pq
    case = cases._case("scores", "decode", 3, q_heads, 1, 1000, min_context=3, dtype=dtype, grouped_angles=True, shuffled_pages=True)
    state = cases.prepare(case, 6)
    want = cases.run(state).clone()
    scores = torch.full((3, q_heads, state["max_seq_len"]), float("nan"), device="cuda:0")
    alone = scores.clone()
    state["out"].zero_()
    pq.pq_decode_attention(state["layout"], state["q"], state["codes"], state["params"], state["v_pool"], state["block_table"],
                           state["seq_lens"], state["max_seq_len"], state["sm_scale"], state["out"], state["workspace"], scores)
    pq.pq_score_keys(state["layout"], state["q"], state["codes"], state["params"], state["block_table"], state["seq_lens"],
                     state["max_seq_len"], alone)
    assert torch.equal(state["out"], want)
    assert torch.equal(scores.nan_to_num(nan=-7.0), alone.nan_to_num(nan=-7.0))
    for s, n in enumerate(cases._lengths(case)):
        assert torch.isnan(alone[s, :, n:]).all() and not torch.isnan(alone[s, :, :n]).any()


@pytest.mark.parametrize("q_heads", [4, 8])
@pytest.mark.parametrize("what", ["radius", "query", "both", "small", "zero_page"])
def test_sizes_far_apart(what, q_heads, monkeypatch):
    """One pair 2^15 times the others in the keys, one element 2^12 times the others in a query, tiny keys, a page of zeros."""
    from perf import cases

    case = cases._case("sizes", "decode", 2, q_heads, 1, 500, grouped_angles=True, dtype="f32")
    keys, queries = cases._keys, cases._queries

    def scaled_keys(case, seed, seq, length):
        k = keys(case, seed, seq, length).clone()
        if what in ("radius", "both"):
            k[..., [7, 71]] *= 3000.0
        if what == "small":
            k *= 2.0 ** -12
        if what == "zero_page":
            k[128:256] = 0.0
        return k

    def scaled_queries(case, seed):
        q = queries(case, seed).clone()
        if what in ("radius", "both"):
            q[..., [7, 71]] *= 1e-5
        if what in ("query", "both"):
            q[..., 20] *= 4096.0
            q[..., 84] *= 1.0 / 4096
        return q * (2.0 ** 12 if what == "small" else 1.0)

    monkeypatch.setattr(cases, "_keys", scaled_keys)
    monkeypatch.setattr(cases, "_queries", scaled_queries)
    state = cases.prepare(case, 8)
    if what in ("query", "both"):
        state["sm_scale"] /= 4096.0
        monkeypatch.setattr(cases.math, "sqrt", lambda x, f=cases.math.sqrt: f(x) * 4096.0 if x == 128 else f(x))
    err = float((cases.run(state).double() - cases.exact(case, 8)).norm() / cases.exact(case, 8).norm())
    print("[sizes]", what, q_heads, err, flush=True)
    assert err <= 6e-6


@pytest.mark.parametrize("shape", [(4, 32, 8, 3000, True), (40, 12, 4, 1000, True), (3, 8, 8, 2000, True), (2, 24, 8, 777, False)], ids=str)
def test_two_stages_and_graph_replay(shape):
    """Partials and merge as two calls, and the call captured in a graph, give the call's result (the two ways of merging
    add the same partials in another order)."""
    from perf import cases

    pq = cases.pq
    seqs, q_heads, kv_heads, context, grouped = shape
    case = cases._case("stages", "decode", seqs, q_heads, kv_heads, context, min_context=context // 2, grouped_angles=grouped)
    state = cases.prepare(case, 4)
    want = cases.run(state).clone()
    pq.pq_decode_partials(state["layout"], state["q"], state["codes"], state["params"], state["v_pool"], state["block_table"],
                          state["seq_lens"], state["max_seq_len"], state["sm_scale"], state["workspace"])
    out = torch.full_like(want, float("nan"))
    pq.pq_decode_merge(state["layout"], seqs, q_heads, state["seq_lens"], state["max_seq_len"], out, state["workspace"])
    assert float((out - want).norm() / want.norm()) <= 1e-6

    stream = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        cases.run(state)
    for turn in range(4):
        state["out"].zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(state["out"], want)
        state["q"].copy_(state["q"].flip(0) if seqs > 1 else -state["q"])      # new inputs are picked up
        want = cases.run(state).clone()
        torch.cuda.synchronize()


@pytest.mark.parametrize("q_heads", [1, 3, 4, 8, 16])
@pytest.mark.parametrize("dtype", ["f16", "f32"])
def test_scores_of_a_tail_without_a_page(q_heads, dtype):
    """The un-quantized keys of the last, incomplete group are scored whatever the block table holds for it: a caller that
    wants scores alone has no packed page there.  Dot products of 128 terms: the bound of the scores, 5e-7."""
    from perf import cases

    pq = cases.pq
    case = cases._case("tail", "serve", 4, q_heads, 1, 600, min_context=130, dtype=dtype, grouped_angles=True, shuffled_pages=True)
    state = cases.prepare(case, 3)
    cases.run(state)                                                      # the new keys are appended
    lens = state["seq_lens"].tolist()
    scores = []
    for entry in (None, -1, state["codes"].shape[0] + 5):
        table = state["block_table"].clone()
        for s, n in enumerate(lens):
            if entry is not None and n % 128:
                table[s, n // 128] = entry
        out = torch.full((4, q_heads, state["max_seq_len"]), float("nan"), device="cuda:0")
        pq.pq_score_keys(state["layout"], state["q"], state["codes"], state["params"], table, state["seq_lens"], state["max_seq_len"],
                         out, state["residual"])
        scores.append(out)
    for out in scores[1:]:
        assert torch.equal(out.nan_to_num(nan=-7.0), scores[0].nan_to_num(nan=-7.0))
    for s, n in enumerate(lens):
        assert not torch.isnan(scores[1][s, :, :n]).any() and torch.isnan(scores[1][s, :, n:]).all()
        tail = n % 128
        if tail:
            want = torch.matmul(state["q"][s].double(), state["residual"][s, 0, :tail].double().t().contiguous())
            assert float((scores[1][s, :, n - tail:n].double() - want).norm() / want.norm()) <= 5e-7


@pytest.mark.parametrize("op,q_heads,dtype", [("score", 3, "f16"), ("score", 8, "f16"), ("decode", 4, "f16"), ("decode", 4, "f32"), ("decode", 8, "f32")])
@pytest.mark.parametrize("tail", [False, True])
def test_one_large_radius_costs_the_others_no_bits(op, q_heads, dtype, tail, monkeypatch):
    """A pair with radii of 15000 beside others of 2^-9, in a pair where the queries are 2^-20 of their largest: products of
    one size.  Bounds as for inputs of one size, 5e-7 for scores and 3e-6 for the output (fp32 arithmetic: 1.3e-7 and 4e-7)."""
    from perf import cases

    pq = cases.pq
    case = cases._case("radius", "serve" if tail else op, 2, q_heads, 1, 500, grouped_angles=True, dtype=dtype)
    keys, queries = cases._keys, cases._queries

    def scaled_keys(case, seed, seq, length):
        k = keys(case, seed, seq, length).float()
        big = 15000.0 * torch.tanh(k[..., [7, 71]])
        k *= 2.0 ** -9
        k[..., [7, 71]] = big
        return k.to(cases._float_dtype(case))

    def scaled_queries(case, seed):
        q = queries(case, seed).float() * 2.0 ** 9
        q[..., [7, 71]] *= 2.0 ** -20
        return q.to(cases._float_dtype(case))

    monkeypatch.setattr(cases, "_keys", scaled_keys)
    monkeypatch.setattr(cases, "_queries", scaled_queries)
    state, want = cases.prepare(case, 12), cases.exact(case, 12)
    got = cases.run(state)
    if tail:                                                              # the new keys are in the residual rows
        got, want = got[0], want[0]
    if tail and op == "score":                                            # the tail's scores, of the sequence that has one
        n = int(state["seq_lens"][1])
        scores = torch.zeros((2, q_heads, state["max_seq_len"]), device="cuda:0")
        pq.pq_score_keys(state["layout"], state["q"], state["codes"], state["params"], state["block_table"], state["seq_lens"],
                         state["max_seq_len"], scores, state["residual"])
        got = scores[1, :, n // 128 * 128:n]
        want = torch.matmul(state["q"][1].double(), state["residual"][1, 0, :n % 128].double().t().contiguous())
    err = float((got.double() - want).norm() / want.norm())
    print("[radius]", op, q_heads, dtype, tail, err, flush=True)
    assert err <= (5e-7 if op == "score" else 3e-6), err
