"""The batched kernel at the edges of its groups: 2, 4 and 8 vectors a group, the last group partly idle,
the smallest hidden size, frames shorter than a step's samples, and subscale lanes whose last-drawn
samples fall inside and outside the context window."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import oracle as O  # noqa: E402
from paper_1802_08435_amd import synth, wavernn  # noqa: E402


def cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


LOGIT = 1e-3    # of a teacher-forced logit (as the scoring tests), and so of h
# of a running sum of the softmax: moving every logit by LOGIT moves it by C (1 - C) 2 LOGIT <= LOGIT / 2,
# and fp32 sums of 256 terms by less than 1e-5
DRAW = LOGIT / 2 + 1e-5


def host(st):
    return {k: st[k].cpu().numpy() for k in ("h", "c", "f")}


def check(w, S, T, frame):
    """One sampling call: the same samples and final state in two pieces, bit for bit; every draw the
    oracle's on the same trajectory, up to a tie at the accuracy of the logits; final state the oracle's.
    Subscale models (which score on the batched kernel): teacher-forced logits and NLL the oracle's."""
    w["frame_len"] = frame
    feat = synth.features(S, T, cond_dim=8, frame_len=frame)
    cond = cuda(feat)
    B = w["B"]
    m = wavernn.Model(w, dtype="bf16", max_streams=S)
    assert m.path(S)[0] == "batched"
    fin = m.new_state(S)
    out = m.sample(T, cond=cond, seed=3, n_streams=S, final=fin)
    st = m.new_state(S)
    if B == 1:
        K = T // 2 + 1                         # off the frames' edges
        two = torch.cat([m.sample(K, cond=cond, seed=3, n_streams=S, final=st).view(torch.int16),
                         m.sample(T - K, cond=cond, seed=3, n_streams=S, init=st, final=st).view(torch.int16)], 1)
    else:
        n = m.schedule_steps(T)
        K = n // 2 + 1
        two = torch.zeros(S, T, dtype=torch.uint16, device="cuda")
        m.sample_steps(two, 0, K, cond=cond, seed=3, final=st)
        m.sample_steps(two, K, n - K, cond=cond, seed=3, init=st, final=st)
        two = two.view(torch.int16)
    m.device_status()
    assert torch.equal(out.view(torch.int16), two)
    tgt, state = out.cpu().numpy(), host(fin)
    for k, v in host(st).items():
        np.testing.assert_array_equal(v, state[k], err_msg=k)
    ref = O.run(O.Weights.from_dict(w, bf16=True), S, T, feat=feat, target=tgt, logits=True, nll=True)
    np.testing.assert_array_equal(state["c"], ref["c"])
    np.testing.assert_array_equal(state["f"], ref["f"])
    assert np.abs(state["h"] - ref["h"]).max() <= LOGIT
    u = np.array([[O.uniforms(3, s * B + n % B, n // B) for n in range(T)] for s in range(S)])   # [S][T][2]
    for i, (z, cls) in enumerate(((ref["zc"], tgt >> 8), (ref["zf"], tgt & 255))):
        C = np.cumsum(np.exp(z.astype(np.float64) - z.max(-1, keepdims=True)), -1)
        C /= C[..., -1:]
        hi = np.take_along_axis(C, cls[..., None].astype(np.int64), -1)[..., 0]
        lo = np.where(cls > 0, np.take_along_axis(C, np.maximum(cls.astype(np.int64) - 1, 0)[..., None], -1)[..., 0], 0.0)
        assert (lo - DRAW <= u[..., i]).all() and (u[..., i] <= hi + DRAW).all()
    if B > 1:
        r = m.score(out, cond=cond)
        m.device_status()
        assert np.abs(r["zc"].cpu().numpy() - ref["zc"]).max() <= LOGIT
        assert np.abs(r["zf"].cpu().numpy() - ref["zf"]).max() <= LOGIT
        assert np.abs(r["nll"].cpu().numpy() - ref["nll"]).max() <= 4 * LOGIT    # two log-softmax terms


@pytest.mark.parametrize("H,S,frame", [(128, 5, 1), (256, 15, 3), (128, 17, 7), (384, 31, 50), (128, 33, 1), (256, 63, 11)])
def test_groups_of_utterances(H, S, frame):
    check(synth.make_weights(H, seed=H + S, cond_dim=8), S, 75, frame)


# F = 0: the sub-tensor before gave the sample just before; B F - 1 inside and past the window's half (16)
@pytest.mark.parametrize("H,S,B,F", [(128, 1, 4, -1), (128, 3, 4, 0), (256, 1, 8, 2), (128, 2, 8, 3), (128, 1, 16, 1),
                                     (128, 2, 16, -1), (128, 4, 16, 1)])
def test_groups_of_lanes(H, S, B, F):
    w = synth.make_weights(H, seed=B + S, cond_dim=8, B=B, ctx_dim=64)
    w["F"] = F
    check(w, S, 24 * B, 3 if B == 4 else 40)
