"""The compiled marshalling of the binding's ordinary calls against the ctypes path: same outputs, same refusals."""
import numpy as np
import pytest

from oracle import approxifer_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.fixture(params=["compiled", "ctypes"])
def binding(request, monkeypatch):
    from paper_2109_09868_amd import binding
    assert binding._marshal()[0] is not None
    if request.param == "ctypes":
        monkeypatch.setattr(binding, "_marshal", lambda: (None, None))
    return binding


def _case():
    import torch
    dev = torch.device("cuda:0")
    K, N, S, A, C, D, G = 3, 12, 2, 1, 7, 33, 5
    rng = np.random.default_rng(3)
    alpha, beta = orc.chebyshev_nodes(K, N)
    t = {"queries": rng.random((G, K, D)), "preds": rng.standard_normal((G, N, C)), "arrival": rng.random((G, N))}
    t = {k: torch.from_numpy(v.astype(np.float32)).to(dev) for k, v in t.items()}
    mask = np.ones((G, N), np.uint8)
    mask[:, 1] = mask[:, 7] = 0
    t["mask"] = torch.from_numpy(mask).to(dev)
    f32, i32 = dict(dtype=torch.float32, device=dev), dict(dtype=torch.int32, device=dev)
    t.update(coded=torch.empty((G, N, D), **f32), out=torch.empty((G, K, C), **f32), status=torch.empty((G,), **i32),
             top1=torch.empty((G, K), **i32), score=torch.empty((G, K), **f32), adv=torch.empty((G, A), **i32),
             made=torch.empty((G, N), dtype=torch.uint8, device=dev), count=torch.empty((G,), **i32))
    return torch, (K, N, S, A, C, D, G), alpha, beta, t


def test_ordinary_calls_reach_the_library(binding):
    torch, (K, N, S, A, C, D, G), alpha, beta, t = _case()
    coded = binding.approxifer_encode(t["queries"], alpha, beta, coded=t["coded"])
    assert coded is t["coded"]
    assert np.allclose(coded.cpu().numpy(), orc.encode(t["queries"].cpu().numpy(), alpha, beta), rtol=0, atol=1e-5)
    Y, m = t["preds"].cpu().numpy(), t["mask"].cpu().numpy()
    ref, _ = orc.decode(Y, m, alpha, beta, S, 1)
    out, status = binding.approxifer_decode(t["preds"], t["mask"], alpha, beta, S, 1, out=t["out"], status=t["status"])
    assert out is t["out"] and status is t["status"] and torch.all(status == 0)
    assert np.allclose(out.cpu().numpy(), ref, rtol=0, atol=1e-5 * np.abs(ref).max())
    for score in (t["score"], None):
        top1, sc, _ = binding.approxifer_decode_top1(t["preds"], t["mask"], alpha, beta, S, 1, top1=t["top1"], score=score,
                                                     status=t["status"], want_score=score is not None)
        assert sc is score and np.array_equal(top1.cpu().numpy(), ref.argmax(2))
        t["top1"].zero_()
        binding.approxifer_top1(out, top1=t["top1"], score=score, want_score=score is not None)
        assert np.array_equal(t["top1"].cpu().numpy(), ref.argmax(2))
    for call in (binding.approxifer_decode_byzantine, binding.approxifer_decode_byzantine_homogeneous):
        given = call(t["preds"], t["mask"], alpha, beta, S, A, 1, out=t["out"], adv=t["adv"], status=t["status"],
                     workspace=binding.NO_WORKSPACE)
        made = call(t["preds"], t["mask"], alpha, beta, S, A, 1)
        assert all(torch.equal(a, b) for a, b in zip(given, made))
    made, count = binding.approxifer_wait_mask(t["arrival"], 4, mask=t["made"], count=t["count"])
    ref_mask, ref_count = orc.wait_mask(t["arrival"].cpu().numpy(), 4)
    assert np.array_equal(made.cpu().numpy(), ref_mask) and np.array_equal(count.cpu().numpy(), ref_count)
    buf = torch.arange(24, dtype=torch.float32, device="cuda:0").view(8, 3)
    groups = binding.approxifer_pad_last_group(buf, 5, 3)
    assert groups.shape == (2, 3, 3) and torch.equal(buf[5], buf[4]) and buf[6, 0] == 18.0
    # a call on another stream than the default is ordered there
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        x = torch.zeros_like(t["preds"])
        torch.cuda._sleep(2000000)
        x.copy_(t["preds"])
        o, _ = binding.approxifer_decode(x, t["mask"], alpha, beta, S, 1, out=torch.empty_like(t["out"]), status=t["status"])
    side.synchronize()
    assert np.allclose(o.cpu().numpy(), ref, rtol=0, atol=1e-5 * np.abs(ref).max())


def test_other_forms_are_taken_and_refused_as_documented(binding):
    torch, (K, N, S, A, C, D, G), alpha, beta, t = _case()

    def decode(**other):
        a = dict(preds=t["preds"], mask=t["mask"], alpha=alpha, beta=beta, S=S, sign_mode=1, out=t["out"], status=t["status"])
        a.update(other)
        return binding.approxifer_decode(**a)

    ref = decode()[0].clone()
    for other in (dict(alpha=list(alpha), beta=tuple(beta)), dict(S=np.int64(S)), dict(alpha=np.asfortranarray(alpha)),
                  dict(beta=np.stack([beta, beta], 1)[:, 0]), dict(stream=torch.cuda.current_stream()), dict(out=None),
                  dict(status=None), dict(alpha=alpha.astype(">f8"))):
        assert torch.equal(decode(**other)[0], ref), other
    wide = torch.empty((G, N, 2 * C), device="cuda:0")
    for error, other in [(TypeError, dict(preds=t["preds"].double())), (TypeError, dict(preds=wide[:, :, :C])),
                         (TypeError, dict(preds=t["preds"].cpu())), (TypeError, dict(mask=t["mask"].bool())),
                         (TypeError, dict(out=t["out"].cpu())), (TypeError, dict(mask=None)),
                         (ValueError, dict(beta=beta[:-1])), (ValueError, dict(out=t["out"][:, :, :-1].contiguous())),
                         (ValueError, dict(status=t["status"][:-1])), (binding.ApproxiferError, dict(S=N)),
                         (binding.ApproxiferError, dict(sign_mode=7))]:
        with pytest.raises(error):
            decode(**other)
    with pytest.raises(Exception):                          # a transform's wrapper has no address
        torch.vmap(lambda p: decode(preds=p)[0])(t["preds"][None])
