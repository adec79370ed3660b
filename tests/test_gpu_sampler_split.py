"""The sampler cuts a row of logits into blocks and only forms the exact noise where a bound says that it can win:
tokens and log-probs against the oracle's choice at vocabularies around the block edges, and for one row, a few rows
and more rows than one block per row would take."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from synth import ModelConfig, make_weights


@pytest.mark.parametrize("vocab,B", [(8, 3), (1023, 1), (1024, 5), (1025, 2), (4097, 1), (5003, 40)])
def test_sampled_tokens_at_block_edges(vocab, B):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_17031_amd as P
    from oracle import neox_oracle as O
    cfg = ModelConfig(1, 64, 4, 16, 4, 128, vocab=vocab, dtype="fp32", pad_id=vocab)
    w = make_weights(cfg, 31, variant="test")
    g = np.random.default_rng(vocab)
    queries = g.integers(1, vocab, size=(B, 4)).astype(np.int32)
    mask = np.ones((B, 4), np.uint8)
    toks, lps, _ = P.Policy(cfg, w).rollout_generate(queries, mask, 7, 0.7, 3)
    lps = lps.cpu().numpy()
    for r in O.verify_rollout(O.OracleModel(w, cfg), toks.cpu().numpy(), mask, 7, 0.7, 3, rows=list(range(B))):
        assert r["token"] == r["argmax"], r
        assert abs(lps[r["row"], r["step"]] - r["logprob"]) <= 1e-4, r
