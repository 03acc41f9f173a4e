"""The smallest calls: contexts whose chunk has five to seven pages (work-groups of eight wavefronts)."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# sequences, query heads, KV heads, longest and shortest context, value bits, query type, bits: at most 256 units, 4 < pages < 8
WIDE = [
    (1, 32, 8, 777, 777, 16, "f16", (4, 4)), (1, 1, 1, 513, 513, 16, "f32", (3, 3)), (5, 40, 5, 895, 1, 16, "f16", (5, 3)),
    (32, 8, 8, 640, 100, 16, "f32", (4, 4)), (3, 32, 2, 768, 129, 16, "f16", (3, 5)), (4, 8, 2, 800, 5, 4, "f16", (4, 4)),
    (4, 14, 2, 641, 300, 2, "f16", (2, 4)), (2, 8, 1, 890, 513, 4, "f32", (3, 3)),
]


@pytest.mark.parametrize("op", ["decode", "serve"])
@pytest.mark.parametrize("shape", WIDE, ids=str)
def test_work_groups_of_eight_wavefronts(shape, op):
    """Bounds as in test_gpu_matrix_attention.py."""
    from perf import cases

    seqs, q_heads, kv_heads, context, shortest, v_bits, dtype, bits = shape
    case = cases._case("wide", op, seqs, q_heads, kv_heads, context, min_context=shortest, v_bits=v_bits, dtype=dtype,
                       r_bits=bits[0], t_bits=bits[1], shuffled_pages=True)
    print("[wide]", op, shape, flush=True)
    state = cases.prepare(case, 7)
    assert cases.pq.pq_decode_merges_in_kernel(state["layout"], seqs, q_heads, state["max_seq_len"], v_bits)
    state["workspace"].fill_(0x5A)
    first = cases.run(state)
    got, want = (first[0], cases.exact(case, 7)[0]) if op == "serve" else (first, cases.exact(case, 7))
    err = float((got.double() - want).norm() / want.norm())
    assert err <= (3e-6 if v_bits == 16 else 4e-5), err
