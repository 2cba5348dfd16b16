"""The single-workgroup fp32 kernel against the oracle over the hidden sizes it serves: the edges of
its padded halves (16, 32 and 36 units), odd halves, frames that change every step, and calls that
continue one another.  Its evaluation order is the oracle's, so samples, state and logits are equal
bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import oracle as O  # noqa: E402
from paper_1802_08435_amd import synth, wavernn  # noqa: E402


def cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("H,S,dc,frame", [(2, 1, 0, 120), (32, 3, 8, 1), (34, 1, 5, 7), (64, 2, 16, 64), (66, 1, 0, 120),
                                          (72, 2, 8, 50)])
def test_small_kernel_is_the_oracle_bit_for_bit(H, S, dc, frame):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    T, K = 200, 67                       # K: off every multiple of 64 and of the frames
    w = synth.make_weights(H, seed=H, cond_dim=dc)
    w["frame_len"] = frame
    feat = synth.features(S, T, cond_dim=dc, frame_len=frame) if dc else None
    cond = None if feat is None else cuda(feat)
    m = wavernn.Model(w, dtype="f32", max_streams=S)
    assert m.path(S)[0] == "single-workgroup"
    st = m.new_state(S)
    a = m.sample(K, cond=cond, seed=9, n_streams=S, final=st)
    b = m.sample(T - K, cond=cond, seed=9, n_streams=S, init=st, final=st)
    out = np.concatenate([a.cpu().numpy(), b.cpu().numpy()], axis=1)
    W = O.Weights.from_dict(w)
    ref = O.run(W, S, T, feat=feat, seed=9)
    np.testing.assert_array_equal(out, ref["out"])
    np.testing.assert_array_equal(st["h"].cpu().numpy(), ref["h"])
    tgt = synth.target_signal(S, T, kind="uniform")
    r = m.score(cuda(tgt), cond=cond)
    m.device_status()
    ref = O.run(W, S, T, feat=feat, target=tgt, logits=True, nll=True)
    np.testing.assert_array_equal(r["zc"].cpu().numpy(), ref["zc"])
    np.testing.assert_array_equal(r["zf"].cpu().numpy(), ref["zf"])
    np.testing.assert_allclose(r["nll"].cpu().numpy(), ref["nll"], rtol=1e-5, atol=1e-5)
    # the NLL alone, and the logits alone, are the same values
    n = m.score(cuda(tgt), cond=cond, logits=False)["nll"]
    z = m.score(cuda(tgt), cond=cond, nll=False)
    m.device_status()
    assert torch.equal(n, r["nll"]) and torch.equal(z["zc"], r["zc"]) and torch.equal(z["zf"], r["zf"])
