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


@pytest.mark.parametrize("kind,mode", [("dense", "global"), ("fused", "thread_local"), ("dense", "relaxed")])
def test_a_captured_call_leaves_other_models_alone(kind, mode):
    """Utterances side by side use internal streams.  While one model's call is captured into a graph,
    another model's call runs at once, and not into the graph; replays give the captured call's samples."""
    make = (lambda s: synth.make_weights(128, seed=s, cond_dim=8)) if kind == "dense" else \
        (lambda s: synth.make_fused_weights(128, F=2, seed=s, cond_dim=8))
    a, b = Call(make(1), 4, 300).alone(), Call(make(2), 3, 240).alone()
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s1):
        g.capture_begin(capture_error_mode=mode)
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


def at_once(calls):
    """Every call on a stream of its own, enqueued one after another."""
    streams = [torch.cuda.Stream() for _ in calls]
    for c in calls:
        c.clear()
    for c, s in zip(calls, streams):
        c.run(s)
    torch.cuda.synchronize()
    for c in calls:
        c.check()


def fused896(seed):
    return synth.make_fused_weights(896, F=2, seed=seed, cond_dim=0)


def test_more_fused_models_than_xcds():
    """A fused grid takes 28 of an XCD's 32 CUs: eight of them run on an XCD each, the ninth waits."""
    at_once([Call(fused896(s), 1, 600).alone() for s in range(9)])


def test_kinds_of_models_beside_each_other():
    """Dense, fused, scoring, subscale, a small model and side-by-side utterances of another dense model."""
    ws = synth.make_weights(256, seed=4, cond_dim=8, B=4, ctx_dim=64)
    ws["F"] = 1
    calls = [Call(synth.make_weights(896, seed=1, cond_dim=8), 1, 700), Call(fused896(2), 2, 600),
             Call(ws, 2, 4 * 300), Call(synth.make_weights(256, seed=3, cond_dim=8), 3, 500),
             Call(synth.make_weights(896, seed=6, cond_dim=8), 1, 650)]
    for c in calls:
        c.alone()
    sc = wavernn.Model(synth.make_weights(896, seed=5, cond_dim=0), max_streams=9)
    tgt = cuda(synth.target_signal(9, 400, seed=2, kind="uniform"))
    one = {S: sc.score(tgt[:S].contiguous(), logits=False)["nll"] for S in (1, 9)}
    sc.device_status()
    s = torch.cuda.Stream()
    for _ in range(3):
        r = {S: sc.score(tgt[:S].contiguous(), logits=False, stream=s)["nll"] for S in (1, 9)}
        at_once(calls)
        sc.device_status(s)
        for S in r:
            assert torch.equal(r[S], one[S])


def test_a_call_that_does_not_fit_waits_for_a_long_one():
    """A batched call that fills every XCD for over two seconds (a bounded wait's limit), and a fused
    call on another stream meanwhile: the second starts when the first has ended."""
    long = Call(synth.make_weights(896, seed=1, cond_dim=0), 64, 400_000)
    short = Call(fused896(2), 1, 1200).alone()
    short.clear()
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    e0, e1, e2 = (torch.cuda.Event(enable_timing=True) for _ in range(3))
    e0.record(s1)
    long.run(s1)
    e1.record(s1)
    short.run(s2)
    e2.record(s2)
    torch.cuda.synchronize()
    assert e0.elapsed_time(e1) > 2000, "the long call must outlast a bounded wait"
    assert e1.elapsed_time(e2) > 0
    long.m.device_status()
    short.check()
