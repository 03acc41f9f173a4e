"""The two ways the arguments of a call are marshalled."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


class Recorder:
    """The native module, and what each of its calls returned."""

    def __init__(self, module):
        self.module, self.made = module, []

    def __getattr__(self, name):
        def call(*args):
            status = getattr(self.module, name)(*args)
            self.made.append((name, status))
            return status
        return call


class Declines:
    def __getattr__(self, name):
        return lambda *a: None


@pytest.mark.parametrize("op,v_bits,calls", [("decode", 16, ["decode_attention"]), ("decode", 2, ["decode_attention"]), ("score", 16, ["score_keys"]),
                                             ("prefill", 4, ["encode_keys", "encode_values"]), ("prefill", 16, ["encode_keys"]),
                                             ("serve", 16, ["append_keys", "decode_attention"]), ("serve", 4, ["append_keys", "decode_attention"])])
def test_both_ways_of_marshalling_make_the_same_call(op, v_bits, calls, monkeypatch):
    """With the native module declining everything the calls go through ctypes; otherwise it makes them all."""
    from perf import cases

    pq = cases.pq
    case = cases._case("both", op, 3, 8, 2, 700, min_context=700 if op == "prefill" else 300, v_bits=v_bits, shuffled_pages=True)
    native = Recorder(pq._marshaller())
    results = []
    for way in (native, Declines()):
        monkeypatch.setattr(pq, "_calls", way)
        result = cases.run(cases.prepare(case, 9))
        results.append(result if isinstance(result, tuple) else (result,))
    assert native.made == [(name, 0) for name in calls]
    for a, b in zip(*results):
        assert torch.equal(a, b)


@pytest.mark.parametrize("v_bits", [16, 4])
def test_scores_and_residual_are_marshalled(v_bits, monkeypatch):
    from perf import cases

    pq = cases.pq
    case = cases._case("all", "serve", 3, 8, 2, 700, min_context=300, v_bits=v_bits, shuffled_pages=True)
    native = Recorder(pq._marshaller())
    results = []
    for way in (native, Declines()):
        monkeypatch.setattr(pq, "_calls", way)
        st = cases.prepare(case, 9)
        cases.run(st)
        scores, alone = torch.full((2, 3, 8, st["max_seq_len"] + 3), -7.0, device="cuda:0")
        pq.pq_decode_attention(st["layout"], st["q"], st["codes"], st["params"], st["v_pool"], st["block_table"], st["seq_lens"], st["max_seq_len"],
                               st["sm_scale"], st["out"], st["workspace"], scores, st["residual"], v_bits, st["v_params"])
        pq.pq_score_keys(st["layout"], st["q"], st["codes"], st["params"], st["block_table"], st["seq_lens"], st["max_seq_len"], alone, st["residual"])
        results.append((st["out"], scores, alone))
    assert native.made == [("append_keys", 0), ("decode_attention", 0), ("decode_attention", 0), ("score_keys", 0)]
    for a, b in zip(*results):
        assert torch.equal(a, b)
    assert torch.equal(results[0][1], results[0][2]) and bool((results[0][1] == -7.0).any())


def test_what_the_native_module_declines_still_works_or_raises():
    from perf import cases

    pq = cases.pq
    state = cases.prepare(cases._case("odd", "decode", 2, 8, 2, 700, min_context=300), 11)
    want = cases.run(state).clone()
    calls = pq._marshaller()
    args = [state[k] for k in ("layout", "q", "codes", "params", "v_pool", "block_table", "seq_lens", "max_seq_len", "sm_scale", "out", "workspace")]
    assert calls.decode_attention(*args, None, None, 16, None) == 0
    for at, odd in ((7, np.int64(state["max_seq_len"])), (8, np.float32(state["sm_scale"])), (1, torch.nn.Parameter(state["q"], requires_grad=False))):
        unusual = list(args)
        unusual[at] = odd
        state["out"].zero_()
        pq.pq_decode_attention(*unusual)
        assert torch.equal(state["out"], want)
    for at, wrong in ((1, state["q"].double()), (1, state["q"].transpose(0, 1)), (2, state["codes"].cpu()), (5, state["block_table"].long()),
                      (6, state["seq_lens"].float()), (4, state["v_pool"][:1]), (9, state["out"].half()), (3, state["params"][:1])):
        bad = list(args)
        bad[at] = wrong
        assert calls.decode_attention(*bad, None, None, 16, None) is None
        with pytest.raises(pq.PolarQuantError):
            pq.pq_decode_attention(*bad)
    with pytest.raises(pq.PolarQuantError, match="workspace"):
        pq.pq_decode_attention(*args[:10], state["workspace"][:256])
    with torch.cuda.stream(torch.cuda.Stream()):                          # torch's current stream, not the default one
        torch.cuda.current_stream().wait_stream(torch.cuda.default_stream())
        state["out"].zero_()
        cases.run(state)
        got = state["out"].clone()
    torch.cuda.synchronize()
    assert torch.equal(got, want)


def test_only_a_layout_is_taken_for_one():
    """Other objects that hold the same bytes raise, as the Python functions do."""
    from perf import cases

    pq = cases.pq
    state = cases.prepare(cases._case("layout", "score", 2, 8, 2, 300), 11)
    args = [state[k] for k in ("q", "codes", "params", "block_table", "seq_lens", "max_seq_len", "scores")]
    calls = pq._marshaller()
    assert calls.score_keys(state["layout"], *args, None) == 0
    for other in (bytes(state["layout"]), bytearray(state["layout"]), memoryview(state["layout"]), None, 7):
        assert calls.score_keys(other, *args, None) is None
        with pytest.raises((AttributeError, TypeError)):
            pq.pq_score_keys(other, *args)

    class Named(pq.Layout):
        pass

    want = state["scores"].clone()
    state["scores"].zero_()
    pq.pq_score_keys(Named(128, 4, 4, 128, 2, 0), *args)
    assert torch.equal(state["scores"], want)
