"""The encoder-side projection at the edges of its tiles: one frame, half a slice of K, rows and
columns that end inside a tile, empty utterances, more than 64 of them (the row tiles are counted 64
utterances at a time), few rows and many (the tile depends on it).  Against a float64 product."""
import numpy as np
import pytest

import synth
from test_gpu_parity import pkg  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,F,J", [(1, 1, 16, 4), (3, 33, 48, 100), (70, 97, 80, 132), (130, 70, 64, 260), (5, 500, 1040, 640)])
@pytest.mark.parametrize("bf16", [False, True])
def test_projection_at_the_edges_of_its_tiles(pkg, B, T, F, J, bf16):  # noqa: F811
    import torch
    dims = synth.ModelDims(F=F, E=8, H=8, L=1, J=J, V1=5)
    model = synth.make_model(dims, 3)
    rng = np.random.default_rng(B + T)
    x = rng.standard_normal((B, T, F)).astype(np.float32)
    ln = rng.integers(0, T + 1, B).astype(np.int32)
    ln[0] = T
    for b in range(B):
        x[b, ln[b]:] = np.nan
    eng = pkg.Engine(model, B, T, flags=pkg.RNNT_FLAG_BF16_ARITHMETIC if bf16 else 0)
    got = eng.encoder_projection(torch.from_numpy(x).cuda(), torch.from_numpy(ln).cuda()).cpu().numpy()
    eng.close()

    def rounded(a):
        return torch.from_numpy(a).bfloat16().double().numpy() if bf16 else a.astype(np.float64)

    w = rounded(model.w_enc)
    for b in range(B):
        want = rounded(x[b, :ln[b]]) @ w.T + model.b_enc
        assert np.allclose(got[b, :ln[b]], want, rtol=1e-5, atol=2e-5), b
        assert not got[b, ln[b]:].any(), "rows beyond enc_len stay untouched"
