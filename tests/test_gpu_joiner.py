"""HIP decoder + joiner + log-softmax (tbs_joiner_logp) against the oracle."""
import numpy as np
import pytest

import oracle
from gpu_util import say
from paper_2211_00484_amd import synth

pytestmark = pytest.mark.gpu

SHAPES = [  # (V, C, sigma, R)
    (16, 32, 0.1, 37),        # Tiny shapes, ragged row count
    (500, 512, 0.05, 70),     # Standard / Graph / Throughput shapes
    (5000, 512, 0.05, 20),    # Large shapes
    (129, 100, 0.3, 33),      # ragged V and C (padding paths)
    # enough rows for the 64 x 128 GEMM tiles (two per compute unit):
    (5000, 512, 0.05, 2100),  # Large shapes, ragged row tile
    (129, 100, 0.3, 16500),   # odd number of 64-column tiles, ragged K and rows
]


@pytest.mark.parametrize("V,C,sigma,R", SHAPES)
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_joiner_matches_oracle(V, C, sigma, R, dtype):
    import torch
    from paper_2211_00484_amd import tbs
    say(f"joiner V={V} C={C} R={R} {dtype}")
    rng = np.random.default_rng(V + C)
    model_np = synth.make_model(rng, V, C, sigma)
    enc = rng.standard_normal((R, C), dtype=np.float32)
    a = rng.integers(0, V, R).astype(np.int32)
    b = rng.integers(0, V, R).astype(np.int32)
    model = tbs.Model.from_synth(model_np, dtype=dtype)
    ctx = torch.from_numpy((a.astype(np.int64) * V + b).astype(np.int32))
    got = tbs.joiner_logp(model, torch.from_numpy(enc).cuda(), ctx).cpu().numpy()
    want = oracle.logp(model_np, enc, a, b, bf16=(dtype == "bf16"))
    err = np.abs(got - want).max()
    say(f"  max |dlogp| = {err:.3g}")
    tol = 1e-4 if dtype == "fp32" else 2e-2
    assert err <= tol
    if dtype == "bf16":  # distance to the exact fp32-operand joiner, for the record
        exact = oracle.logp(model_np, enc, a, b, bf16=False)
        say(f"  bf16 vs fp32-operand oracle: {np.abs(got - exact).max():.3g}")


def test_joiner_empty_batch():
    import torch
    from paper_2211_00484_amd import tbs
    model = tbs.Model.from_synth(synth.make_model(np.random.default_rng(0), 8, 16, 0.1))
    out = tbs.joiner_logp(model, torch.zeros((0, 16), device="cuda"), torch.zeros(0, dtype=torch.int32))
    assert out.shape == (0, 8)


# Batches large enough for the 256 x 256 bf16 tiles (at least four per compute unit),
# checked on sampled rows (every row is independent): the first and last row tiles,
# the ragged tail and random rows in between.
WIDE = [  # (V, C, sigma, R)
    (5000, 512, 0.05, 256 * 53 + 77),   # Large shapes: 54 x 20 tiles, ragged rows
    (999, 300, 0.3, 256 * 256 + 5),     # partial last vocabulary tile, ragged K
]


@pytest.mark.parametrize("V,C,sigma,R", WIDE)
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_joiner_large_batches_sampled_rows(V, C, sigma, R, dtype):
    import torch
    from paper_2211_00484_amd import tbs
    say(f"joiner (large batch) V={V} C={C} R={R} {dtype}")
    rng = np.random.default_rng(V + C + R)
    model_np = synth.make_model(rng, V, C, sigma)
    enc = rng.standard_normal((R, C), dtype=np.float32)
    a = rng.integers(0, V, R).astype(np.int32)
    b = rng.integers(0, V, R).astype(np.int32)
    model = tbs.Model.from_synth(model_np, dtype=dtype)
    ctx = torch.from_numpy((a.astype(np.int64) * V + b).astype(np.int32))
    got = tbs.joiner_logp(model, torch.from_numpy(enc).cuda(), ctx).cpu().numpy()
    idx = np.unique(np.concatenate([np.arange(300), np.arange(R - 300, R),
                                    rng.integers(0, R, 400)]))
    want = oracle.logp(model_np, enc[idx], a[idx], b[idx], bf16=(dtype == "bf16"))
    err = np.abs(got[idx] - want).max()
    say(f"  max |dlogp| over {len(idx)} rows = {err:.3g}")
    assert err <= (1e-4 if dtype == "fp32" else 2e-2)
    assert np.isfinite(got).all()


# Edges of the joiner's tilings: sweep (C <= 512, at least one 16 x 64 tile per compute unit;
# 128 or 256 columns a workgroup, groups of 16-row blocks), GEMM tiles with few and with
# ragged column tiles, small tiles with K beyond one chunk.
TILES = [  # (V, C, R)
    (500, 512, 600), (60, 512, 4200), (64, 500, 4097), (65, 33, 2113), (129, 512, 1366),
    (513, 511, 500), (2, 8, 4100), (1000, 512, 256), (5000, 512, 300),
    (200, 512, 16390), (641, 512, 6145),
    (1000, 768, 1000), (300, 1025, 130), (2000, 640, 2100),
]


@pytest.mark.parametrize("V,C,R", TILES)
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_joiner_tilings(V, C, R, dtype):
    import torch
    from paper_2211_00484_amd import tbs
    say(f"joiner tiling V={V} C={C} R={R} {dtype}")
    rng = np.random.default_rng(V * 31 + C + R)
    model_np = synth.make_model(rng, V, C, 0.1)
    enc = rng.standard_normal((R, C), dtype=np.float32)
    a = rng.integers(0, V, R).astype(np.int32)
    b = rng.integers(0, V, R).astype(np.int32)
    model = tbs.Model.from_synth(model_np, dtype=dtype)
    ctx = torch.from_numpy((a.astype(np.int64) * V + b).astype(np.int32))
    got = tbs.joiner_logp(model, torch.from_numpy(enc).cuda(), ctx).cpu().numpy()
    idx = np.unique(np.concatenate([np.arange(min(R, 40)), np.arange(max(0, R - 40), R),
                                    rng.integers(0, R, 200)]))
    want = oracle.logp(model_np, enc[idx], a[idx], b[idx], bf16=(dtype == "bf16"))
    # fp32: tanh and products to 2e-7 each over C terms of |w| ~ 0.1; bf16: a tanh that
    # rounds to its neighbour (2^-9) now and then
    assert np.abs(got[idx] - want).max() <= (2e-5 if dtype == "fp32" else 2e-2)
    assert np.isfinite(got).all()


def _logp64(m, enc, a, b):
    """Log-probabilities in float64, the joiner input's tanh included."""
    dec = np.maximum(m.conv[:, 0] * m.embed[a].astype(np.float64) + m.conv[:, 1] * m.embed[b], 0)
    with np.errstate(over="ignore", invalid="ignore"):
        z = np.tanh(enc + dec) @ m.w_out.astype(np.float64).T + m.b_out.astype(np.float64)
    top = z.max(1, keepdims=True)
    return z - (top + np.log(np.exp(z - top).sum(1, keepdims=True)))


def _logp_gpu(m, enc, a, b, dtype="fp32"):
    import torch
    from paper_2211_00484_amd import tbs
    model = tbs.Model.from_synth(m, dtype=dtype)
    ctx = torch.from_numpy((a * m.vocab_size + b).astype(np.int32))
    return tbs.joiner_logp(model, torch.from_numpy(enc).cuda(), ctx).cpu().numpy()


# fp32 logits: tanh to 2e-7 absolute, operands and products to 2^-22, sums of C terms; per
# unit of a label's own largest weight, as random signs add (the factor 3: worst of the rows)
LOGIT_EPS = 3 * (2e-7 + 2.0 ** -22)

# every tiling: small tiles, sweep, 64 x 128, and K beyond 512 in small and in large tiles
RANGE_SHAPES = [(100, 64, 50), (500, 512, 40), (500, 512, 700), (700, 500, 9000), (300, 600, 40), (2000, 768, 2100)]


@pytest.mark.parametrize("scale", [0.0, 1e-37, 1e-12, 1.0, 1e6, 1e30])
@pytest.mark.parametrize("V,C,R", [(100, 64, 50), (100, 64, 2600), (700, 64, 3000), (300, 600, 40)])
def test_joiner_weight_scales(scale, V, C, R):
    """fp32 weights of any magnitude, rows 2^0 ... 2^-30 of the largest: finite, and right to
    fp32's accuracy in each label's logit and in the normaliser (which the largest labels
    set; what the small labels keep beside large ones is test_joiner_weight_range's)."""
    rng = np.random.default_rng(3)
    m = synth.make_model(rng, V, C, 1.0)
    m.w_out *= (np.float32(scale) * 2.0 ** -rng.integers(0, 31, size=(V, 1))).astype(np.float32)
    m.b_out[:] = 0
    enc = rng.standard_normal((R, C), dtype=np.float32)
    a, b = rng.integers(0, V, R), rng.integers(0, V, R)
    got, want = _logp_gpu(m, enc, a, b), _logp64(m, enc, a, b)
    eps = LOGIT_EPS * np.sqrt(C) * np.abs(m.w_out).max(1)
    tol = 1e-6 + 2e-7 * np.abs(want) + eps + (np.exp(want) * eps).sum(1, keepdims=True)
    assert (np.abs(got - want) <= tol).all()


@pytest.mark.parametrize("p", [0, 20, 24, 27, 40, 100])
@pytest.mark.parametrize("where", ["row", "column"])
@pytest.mark.parametrize("V,C,R", RANGE_SHAPES)
def test_joiner_weight_range(V, C, R, where, p):
    """Weights 2^p above the others that no other label's result depends on: a label's row,
    the label masked by its bias, or the column of a unit whose input is 0.  The others keep
    fp32's accuracy."""
    rng = np.random.default_rng(V + C)
    m = synth.make_model(rng, V, C, 0.05)
    enc = rng.standard_normal((R, C), dtype=np.float32)
    a, b = rng.integers(0, V, R), rng.integers(0, V, R)
    own = np.abs(m.w_out).max()
    if where == "row":
        m.w_out[3] *= np.float32(2.0 ** p)
        m.b_out[3] = -3e38
    else:
        m.w_out[:, 7] = np.float32(0.05 * 2.0 ** p)
        m.embed[:, 7] = 0
        enc[:, 7] = 0
    got, want = _logp_gpu(m, enc, a, b), _logp64(m, enc, a, b)
    keep = np.arange(V) != (3 if where == "row" else -1)
    err = np.abs(got - want)[:, keep].max()
    say(f"  {where} 2^{p}: max |dlogp| = {err:.3g}")
    assert err <= 2e-7 * np.abs(want[:, keep]).max() + 2 * LOGIT_EPS * np.sqrt(C) * own


@pytest.mark.parametrize("V,C,R", RANGE_SHAPES)
def test_joiner_infinite_weight(V, C, R):
    """A weight of minus infinity on a positive unit makes its label impossible and leaves
    the others alone."""
    rng = np.random.default_rng(V + C + 1)
    m = synth.make_model(rng, V, C, 0.05)
    enc = rng.standard_normal((R, C), dtype=np.float32)
    a, b = rng.integers(0, V, R), rng.integers(0, V, R)
    own = np.abs(m.w_out).max()
    m.w_out[3, 7] = -np.inf
    m.embed[:, 7] = 0
    enc[:, 7] = rng.uniform(0.1, 2.0, R)
    got = _logp_gpu(m, enc, a, b)
    keep = np.arange(V) != 3
    m.w_out[3, 7] = 0
    m.b_out[3] = -3e38
    want = _logp64(m, enc, a, b)
    assert (got[:, 3] == -np.inf).all()
    assert np.abs(got - want)[:, keep].max() <= (2e-7 * np.abs(want[:, keep]).max() +
                                                 2 * LOGIT_EPS * np.sqrt(C) * own)


@pytest.mark.parametrize("V,C,R", [(500, 512, 512), (500, 512, 3000), (1000, 512, 300)])
def test_joiner_bf16_sum_error(V, C, R):
    """The sums over C of the bf16 sweep at large logits, where they set the error (the
    median, so that the few tanh that round to a neighbouring bf16 value do not count).  With
    16 products of 32 in chains of four the median is 7.8e-7 to 8.1e-7, in chains of eight,
    whose partial sums are larger, 9.1e-7 to 9.4e-7."""
    rng = np.random.default_rng(V + R)
    m = synth.make_model(rng, V, C, 0.5)
    enc = rng.standard_normal((R, C), dtype=np.float32)
    a, b = rng.integers(0, V, R), rng.integers(0, V, R)
    got = _logp_gpu(m, enc, a, b, dtype="bf16")
    want = oracle.logp(m, enc, a.astype(np.int32), b.astype(np.int32), bf16=True)
    med = np.median(np.abs(got - want))
    say(f"  median |dlogp| = {med:.3g}")
    assert med <= 8.6e-7
