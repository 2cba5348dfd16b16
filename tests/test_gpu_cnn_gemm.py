"""The conditioning CNN's GEMMs at the edges of their tiles: row counts around 64, 96 and 128 and around
the switch between one workgroup per tile and one per group of the K loop, taps past the utterance's end,
several utterances, residual and convolution widths that differ and exceed a workgroup's threads.  Against the
oracle's network."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import oracle as O  # noqa: E402
from paper_1802_08435_amd import synth, wavernn  # noqa: E402


@pytest.mark.parametrize("rows,S,Rc,Cc,layers", [(1, 1, 128, 128, 10), (16, 1, 256, 128, 2), (25, 1, 128, 256, 3),
                                                 (33, 2, 640, 128, 2), (260, 1, 768, 128, 2), (1000, 1, 128, 128, 2),
                                                 (5500, 1, 128, 128, 1), (30, 1, 512, 1152, 1), (9, 1, 1152, 1408, 2)])
def test_cnn_rows_against_the_oracle(rows, S, Rc, Cc, layers):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B, Dx = 4, 128
    w = synth.make_weights(128, seed=1, cond_dim=0, B=B, ctx_dim=Dx)
    w["F"] = 124
    w["cnn"] = synth.make_cnn_weights(B, Rc=Rc, Cc=Cc, Dx=Dx, layers=layers, seed=rows)
    m = wavernn.Model(w, max_streams=S)
    seq = synth.target_signal(S, rows * B, seed=rows, kind="uniform")
    out = m.ctx_cnn(torch.from_numpy(seq).cuda()).cpu().numpy()
    m.device_status()
    bf = {k: (O.bf16_round(v) if isinstance(v, np.ndarray) else v) for k, v in w["cnn"].items()}
    for u in range(S):
        for s in range(B):
            ref = O.ctx_cnn(bf, seq[u], s)
            # each product carries about 2^-16 of its activation: 6e-5 of the largest value through ten layers
            assert np.abs(out[u, s] - ref).max() <= 6e-5 * max(1.0, np.abs(ref).max()), (u, s)
