"""What the serving loop does on the host: the checks of a step's arguments and the objects that it hands out.  The library's
calls are replaced by stand-ins that record the shapes they were given, so no GPU is needed."""
import pytest
import torch

from paper_2109_09868_amd import binding, serving

K, N, S, D, C, MAX_Q = 4, 6, 1, 5, 3, 21


@pytest.fixture
def loop(monkeypatch):
    calls = []

    def record(name):
        def call(*args, **kw):
            tensors = [t for t in list(args) + list(kw.values()) if isinstance(t, torch.Tensor)]
            calls.append((name, [tuple(t.shape) for t in tensors]))
            return {"encode": kw.get("coded"), "wait_mask": (kw.get("mask"), kw.get("count"))}.get(name)
        return call

    real_pad = binding.approxifer_pad_last_group

    def pad(buffer, Q, K, stream=None):
        G = binding.approxifer_group_count(Q, K)
        if G < 0 or buffer.shape[0] < G * K:
            return real_pad(buffer, Q, K)                # raises
        return buffer[: G * K].view(G, K, -1)

    monkeypatch.setattr(binding, "approxifer_pad_last_group", pad)
    for name in ("encode", "wait_mask", "decode", "decode_top1", "top1"):
        monkeypatch.setattr(binding, "approxifer_" + name, record(name))
    lp = serving.ServingLoop(K, N, S, 0, D, C, MAX_Q, "cpu")
    lp.calls = calls
    return lp


def _step(loop, Q, model=None, **kw):
    loop.calls.clear()
    arrival = torch.zeros((loop.max_groups, N))
    return loop.step(Q, model or (lambda x: x[:, :C]), arrival, **kw)


@pytest.mark.parametrize("Q", [-1, -1000, MAX_Q + 4, 10 ** 6])
def test_a_stream_that_the_buffer_cannot_hold_is_a_value_error(loop, Q):
    with pytest.raises(ValueError):
        _step(loop, Q)
    assert loop.calls == []


@pytest.mark.parametrize("want_values", [True, False])
def test_what_a_step_hands_out_is_the_callers_own(loop, want_values):
    first = None
    for Q in (21, 21, 20, 9, 21):                        # the same length again, and others in between
        G = -(-Q // K)
        reshaped = []

        def model(rows):
            assert rows.shape == (G * N, D)
            y = rows[:, :C].clone()
            reshaped.append(rows.unsqueeze_(0))
            return y

        res = _step(loop, Q, model, tamper=lambda p: reshaped.append(p.resize_(3, 2)), want_values=want_values)
        shapes = {"top1": (Q,), "mask": (G, N), "status": (G,), "coded": (G, N, D), "preds": (G, N, C), "adv": (G, 0)}
        if want_values:
            shapes["values"] = (Q, C)
        assert {k: tuple(res[k].shape) for k in shapes} == shapes and (want_values or res["values"] is None)
        assert res["groups"] == G
        if first is None:
            first = list(loop.calls)
        elif Q == 21:
            assert loop.calls == first                   # the calls see the shapes they saw before
        for buf, key in ((loop.mask, "mask"), (loop.preds, "preds"), (loop.coded, "coded"), (loop.status, "status")):
            assert res[key].data_ptr() == buf.data_ptr()                      # views of the loop's buffers
        for t in res.values():
            if isinstance(t, torch.Tensor):
                t.unsqueeze_(0)
                t.resize_(0)                             # in place, as a caller may


def test_a_buffer_put_in_place_of_another_is_the_one_used(loop):
    _step(loop, MAX_Q)
    loop.preds = torch.full_like(loop.preds, 7.0)
    res = _step(loop, MAX_Q, lambda x: torch.ones((x.shape[0], C)))
    assert res["preds"].data_ptr() == loop.preds.data_ptr() and bool((loop.preds == 1.0).all())
