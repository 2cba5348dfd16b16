"""Scoring at the edges of its groups: 1, 2, 4 and 8 utterances a group, the last group partly used, short
utterances around the batches of targets, frames of odd length.  Every utterance's logits and NLL are those
of scoring it alone, bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import oracle as O  # noqa: E402
from paper_1802_08435_amd import synth, wavernn  # noqa: E402


def cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("H,S,T,frame", [(128, 8, 1, 1), (128, 9, 64, 7), (256, 17, 65, 64), (384, 31, 129, 63),
                                         (512, 1, 66, 200), (896, 33, 66, 200), (128, 64, 130, 3)])
def test_groups_equal_one_at_a_time(H, S, T, frame):
    w = synth.make_weights(H, seed=S, cond_dim=8)
    w["frame_len"] = frame
    feat = synth.features(S, T, cond_dim=8, frame_len=frame, per_stream_seed=True)
    tgt = synth.target_signal(S, T, seed=3, kind="uniform")
    m, one = wavernn.Model(w, max_streams=S), wavernn.Model(w)
    many = m.score(cuda(tgt), cond=cuda(feat))
    m.device_status()
    for s in sorted({0, 1, S // 2, S - 2, S - 1} & set(range(S))):
        r = one.score(cuda(tgt[s:s + 1]), cond=cuda(feat[s:s + 1]))
        one.device_status()
        for k in ("zc", "zf", "nll"):
            assert torch.equal(r[k][0], many[k][s]), (k, s)
    assert not any(torch.isnan(many[k]).any() for k in many)
    ref = O.run(O.Weights.from_dict(w, bf16=True), 1, T, feat=feat[:1], target=tgt[:1], logits=True)
    assert np.abs(many["zc"][0].cpu().numpy() - ref["zc"][0]).max() <= 1e-3
    assert np.abs(many["zf"][0].cpu().numpy() - ref["zf"][0]).max() <= 1e-3


def test_one_frame_a_sample_over_half_a_million_frames():
    """More than 2^16 groups of 8 frames in one call: frames of one sample with repeated features score as
    longer frames do."""
    T, L = 525_000, 50
    w = synth.make_weights(128, seed=4, cond_dim=4)
    feat = synth.features(1, T, cond_dim=4, frame_len=L)
    tgt = cuda(synth.target_signal(1, T, seed=3, kind="uniform"))
    nll = {}
    for n in (L, 1):
        w["frame_len"] = n
        f = np.repeat(feat, L // n, axis=1)
        assert f.shape[1] * n == T and (n > 1 or f.shape[1] > 8 * 65536)
        m = wavernn.Model(w)
        nll[n] = m.score(tgt, cond=cuda(f), logits=False)["nll"]
        m.device_status()
        m.close()
    assert torch.equal(nll[1], nll[L])
