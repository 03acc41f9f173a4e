"""Attention launches that try the cut whose chunks all start at once and then have the general rule's chunks or the host's, in the
grid and the workspace that were sized for the former (tests/test_cut_host.py says which gets which).  Against float64; the
same bits on a second call.  Bounds as in test_gpu_resident_cut.py."""
import pytest

torch = pytest.importorskip("torch")

from test_cut_host import FALLBACKS  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,kv_heads,group,bound,v_bits,grouped", [f[:-1] for f in FALLBACKS])
def test_every_chunk_is_taken(monkeypatch, lens, kv_heads, group, bound, v_bits, grouped):
    from perf import cases

    import paper_2502_00527_amd as pq

    monkeypatch.setattr(cases, "_lengths", lambda case: lens)
    case = cases._case("fallback", "decode", len(lens), kv_heads * group, kv_heads, max(lens), min_context=min(lens), v_bits=v_bits, shuffled_pages=True,
                       grouped_angles=grouped)
    print("[cut fallbacks]", case, bound, flush=True)
    state = cases.prepare(case, 5)
    pages = (bound + 127) // 128
    state["block_table"] = torch.nn.functional.pad(state["block_table"], (0, pages - state["block_table"].shape[1])).contiguous()
    state["max_seq_len"] = bound
    state["workspace"] = torch.empty(pq.pq_decode_workspace_bytes(state["layout"], len(lens), kv_heads * group, bound), dtype=torch.uint8, device="cuda:0")
    assert pq.pq_decode_merges_in_kernel(state["layout"], len(lens), kv_heads * group, bound, v_bits)
    got, want = cases.run(state).clone(), cases.exact(case, 5)
    bound_of_one = 1e-4 if v_bits != 16 else (1.2e-5 if grouped else 4e-6)
    for s, n in enumerate(lens):
        err = float((got[s].double() - want[s]).norm() / want[s].norm())
        assert err <= bound_of_one, (s, n, err)
    assert torch.equal(got, cases.run(state))
