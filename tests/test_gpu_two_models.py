"""Calls of several models that overlap on one device: separate models are independent, and each call's
samples, states and scores are those of the call made alone, bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1802_08435_amd import synth, wavernn  # noqa: E402


def cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


class Call:
    """One sampling call with its own buffers, made on a given stream."""

    def __init__(self, w, S, T, seed=5, max_streams=None):
        self.m = wavernn.Model(w, max_streams=max_streams or S)
        self.S, self.T, self.seed = S, T, seed
        self.cond = None if w.get("Wc") is None else cuda(synth.features(S, T, cond_dim=w["Wc"].shape[1], seed=seed))
        self.out = torch.zeros(S, T, dtype=torch.uint16, device="cuda")
        self.fin = self.m.new_state(S)

    def run(self, stream=None):
        self.m.sample(self.T, cond=self.cond, seed=self.seed, n_streams=self.S, out=self.out, final=self.fin,
                      stream=stream)
        return self

    def result(self):
        return [self.out.cpu().numpy().copy()] + [self.fin[k].cpu().numpy().copy() for k in ("h", "c", "f")]

    def alone(self):
        torch.cuda.synchronize()
        self.run()
        self.m.device_status()
        self.ref = self.result()
        self.clear()
        return self

    def clear(self):
        self.out.zero_()
        self.fin["h"].zero_()
        torch.cuda.synchronize()

    def check(self):
        self.m.device_status()
        for a, b in zip(self.result(), self.ref):
            np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("kind", ["dense", "fused"])
def test_a_captured_call_leaves_other_models_alone(kind):
    """Utterances side by side use internal streams.  While one model's call is captured into a graph,
    another model's call runs at once, and not into the graph; replays give the captured call's samples."""
    make = (lambda s: synth.make_weights(128, seed=s, cond_dim=8)) if kind == "dense" else \
        (lambda s: synth.make_fused_weights(128, F=2, seed=s, cond_dim=8))
    a, b = Call(make(1), 4, 300).alone(), Call(make(2), 3, 240).alone()
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s1):
        g.capture_begin(capture_error_mode="relaxed")
        try:
            a.run(s1)
            b.run(s2)
        finally:
            g.capture_end()
    torch.cuda.synchronize()
    b.check()
    assert not a.out.cpu().numpy().any()                       # captured, not run
    for _ in range(3):
        b.clear()
        a.clear()
        g.replay()
        torch.cuda.synchronize()
        a.check()
        assert not b.out.cpu().numpy().any()
        b.run()                                  # eager calls between replays, on the same internal streams
        b.check()
        a.run()
        a.check()
