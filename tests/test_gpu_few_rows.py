"""Decode passes of few sequences: sampled tokens and log-probs against the oracle for batches at the edges of the row
tiles (16, 32, 48, 64, 128, 256 and one past), every head size of the single-query attention kernel, contexts shorter and longer
than what one block takes in one go, both modes, and column counts that are no multiple of a block's columns."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from synth import ModelConfig, make_weights

TOL = {"fp32": 1e-4, "bf16": 2e-2}  # the library's bars for log-probs
NEAR_TIE = 1e-2

# (d_model, heads, head_dim, rotary, d_ff, vocab)
SHAPES = {
    "hd16": (128, 8, 16, 4, 192, 211), "hd64": (128, 2, 64, 16, 512, 1003), "hd80": (320, 4, 80, 20, 448, 517),
    "hd128": (256, 2, 128, 32, 320, 300), "hd256": (256, 1, 256, 64, 1024, 259),
}


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("shape,B,lo,hi", [
    ("hd64", 1, 1, 1), ("hd80", 1, 300, 300), ("hd16", 15, 1, 40), ("hd256", 16, 5, 90), ("hd80", 17, 1, 70),
    ("hd128", 32, 3, 33), ("hd64", 33, 1, 130), ("hd80", 48, 60, 61), ("hd16", 49, 1, 9), ("hd64", 64, 1, 20),
    ("hd128", 64, 1, 8), ("hd64", 65, 1, 8), ("hd80", 128, 1, 40), ("hd256", 129, 1, 9), ("hd16", 193, 1, 70),
    ("hd80", 256, 1, 8), ("hd64", 257, 1, 8)])
def test_decode_of_few_sequences(dtype, shape, B, lo, hi):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_17031_amd as P
    from oracle import neox_oracle as O
    d, H, hd, r, F, V = SHAPES[shape]
    cfg = ModelConfig(2, d, H, hd, r, F, vocab=V, dtype=dtype, pad_id=V)
    w = make_weights(cfg, 77, variant="test")
    g = np.random.default_rng(B)
    lens = g.integers(lo, hi + 1, size=B)
    lens[0], lens[-1] = lo, hi
    mask = (np.arange(hi)[None, :] >= (hi - lens)[:, None]).astype(np.uint8)
    queries = np.where(mask == 1, g.integers(1, V, size=(B, hi)), V).astype(np.int32)
    N = 4
    toks, lps, _ = P.Policy(cfg, w).rollout_generate(queries, mask, 11, 0.7, N)
    lps = lps.cpu().numpy()
    rows = sorted({0, B // 2, B - 1})
    for rep in O.verify_rollout(O.OracleModel(w, cfg), toks.cpu().numpy(), mask, 11, 0.7, N, rows=rows):
        assert rep["deficit"] <= (0.0 if dtype == "fp32" else NEAR_TIE), rep
        assert abs(lps[rep["row"], rep["step"]] - rep["logprob"]) <= TOL[dtype], rep
