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


@pytest.mark.parametrize("B,T,F,J", [(2, 40, 1040, 68), (2, 40, 272, 68), (40, 70, 112, 1028)])
def test_projection_of_frames_and_weights_of_very_different_magnitude(pkg, B, T, F, J):  # noqa: F811
    """fp32 frames and weights are split into fp16 parts after a power of two of the row, a frame's from its first 32
    values: rows that grow, rows of zeros up to there, tiny and huge rows.  A part below fp16's normal range is off by
    2^-25, so a value by 2^-37 of a frame's largest and by 2^-39 of a column's; sums of K products by K 2^-24 of
    their magnitudes."""
    import torch
    model = synth.make_model(synth.ModelDims(F=F, E=8, H=8, L=1, J=J, V1=5), 3)
    rng = np.random.default_rng(B + F)
    x = rng.standard_normal((B, T, F)).astype(np.float32)
    x[:, 1::8] *= np.exp2(np.linspace(-30, 30, F)).astype(np.float32)
    x[:, 2::8, :40] = 0.0
    x[:, 3::8] *= np.float32(2.0 ** -110)
    x[:, 4::8] *= np.float32(2.0 ** 100)
    x[:, 5::8, F - 1] = 1e6
    x[:, 6::8, :] = 0.0
    model.w_enc *= np.exp2(rng.integers(-20, 12, J)).astype(np.float32)[:, None]
    model.b_enc[:] = 0.0
    ln = np.full(B, T, np.int32)
    eng = pkg.Engine(model, B, T)
    got = eng.encoder_projection(torch.from_numpy(x).cuda(), torch.from_numpy(ln).cuda()).cpu().numpy()
    eng.close()
    x, w = x.astype(np.float64), model.w_enc.astype(np.float64)
    want, size = x @ w.T, np.abs(x) @ np.abs(w).T
    bound = (F + 4) * (2.0 ** -24 * size + 2.0 ** -36 * np.abs(x).max(-1, keepdims=True) * np.abs(w).max(-1))
    assert (np.abs(got - want) <= bound + 1e-37).all()


@pytest.mark.parametrize("B,T,F,J", [(2, 40, 1040, 68), (2, 40, 272, 68), (40, 70, 112, 1028)])
@pytest.mark.parametrize("size", [1e5, 1e7, 1e12])
@pytest.mark.parametrize("at", [5, -1])
def test_projection_of_frames_with_one_large_feature(pkg, B, T, F, J, at, size):  # noqa: F811
    """A feature far larger than the others, whose weights are that much smaller, or zero: sums as accurate as fp32
    products are, K 2^-24 of their magnitudes."""
    import torch
    model = synth.make_model(synth.ModelDims(F=F, E=8, H=8, L=1, J=J, V1=5), 3)
    rng = np.random.default_rng(B + F)
    x = rng.standard_normal((B, T, F)).astype(np.float32)
    x[:, ::3, at] *= np.float32(size)
    model.w_enc[:, at] /= np.float32(size)
    model.w_enc[::2, at] = 0.0
    ln = np.full(B, T, np.int32)
    eng = pkg.Engine(model, B, T)
    got = eng.encoder_projection(torch.from_numpy(x).cuda(), torch.from_numpy(ln).cuda()).cpu().numpy()
    eng.close()
    x, w = x.astype(np.float64), model.w_enc.astype(np.float64)
    bound = (F + 4) * 2.0 ** -24 * (np.abs(x) @ np.abs(w).T + np.abs(model.b_enc))
    assert (np.abs(got - (x @ w.T + model.b_enc)) <= bound).all()


@pytest.mark.parametrize("B,T,F,J", [(2, 40, 1040, 68), (2, 40, 272, 68), (40, 70, 112, 1028)])
@pytest.mark.parametrize("where", ["frames", "weights"])
def test_projection_of_values_that_are_not_finite(pkg, B, T, F, J, where):  # noqa: F811
    """Infinities and NaN come out where the fp32 product has them, and the rest as ever."""
    import torch
    model = synth.make_model(synth.ModelDims(F=F, E=8, H=8, L=1, J=J, V1=5), 3)
    rng = np.random.default_rng(B + F)
    x = rng.standard_normal((B, T, F)).astype(np.float32)
    if where == "frames":
        x[0, 3, 5], x[1, 39, F - 1], x[0, 35, 50], x[1, 7, 1] = np.inf, -np.inf, 3.4e38, np.nan
    else:
        model.w_enc[1, 3], model.w_enc[66, F - 1] = np.inf, -np.inf
    ln = np.full(B, T, np.int32)
    eng = pkg.Engine(model, B, T)
    got = eng.encoder_projection(torch.from_numpy(x).cuda(), torch.from_numpy(ln).cuda()).cpu().numpy()
    eng.close()
    with np.errstate(invalid="ignore", over="ignore"):
        want = x.astype(np.float64) @ model.w_enc.T.astype(np.float64) + model.b_enc
        want = np.where(np.abs(want) > 3.4e38, np.copysign(np.inf, want), want)
    assert (np.isnan(got) == np.isnan(want)).all()
    fine = np.isfinite(want)
    assert (got[np.isinf(want)] == want[np.isinf(want)]).all()
    assert np.allclose(got[fine], want[fine], rtol=1e-5, atol=2e-5)
