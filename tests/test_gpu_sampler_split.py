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


def _model_with_logits(value, rows, vocab):
    """A model whose logits of the tokens in `rows` are `value` at every step: coordinate 0 of the final LayerNorm's
    output is 1, and those rows of the output embedding hold `value` there."""
    cfg = ModelConfig(1, 64, 4, 16, 4, 128, vocab=vocab, dtype="fp32", pad_id=vocab)
    w = make_weights(cfg, 31, variant="test")
    w["lnf_g"][0], w["lnf_b"][0] = 0, 1
    w["embed_out"][rows, 0] = value
    return cfg, w


@pytest.mark.parametrize("value", [np.nan, -np.inf])
@pytest.mark.parametrize("rows,vocab,B", [
    (slice(2002, 5003), 5003, 2), (slice(0, 1024), 5003, 600), (slice(0, 300), 1025, 1), (slice(7, 8), 4097, 3)])
def test_logits_that_are_not_finite(value, rows, vocab, B):
    """Whole blocks and whole threads without a finite logit, and single ones.  A NaN shows in the log-prob of every
    token of its row; a logit of -inf is a token of probability 0.  Neither is sampled."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_17031_amd as P
    from oracle import neox_oracle as O
    cfg, w = _model_with_logits(value, rows, vocab)
    g = np.random.default_rng(vocab)
    queries = g.integers(1, vocab, size=(B, 4)).astype(np.int32)
    toks, lps, _ = (x.cpu().numpy() for x in P.Policy(cfg, w).rollout_generate(queries, np.ones((B, 4), np.uint8), 7, 0.7, 3))
    _, w0 = _model_with_logits(0.0, rows, vocab)
    m = O.OracleModel(w0, cfg)
    for b in sorted({0, B // 2, B - 1}):
        x, _ = O.forward_sequence(m, toks[b], np.arange(7))
        logits, _ = O.heads(m, x[3:-1])
        logits[:, rows] = -np.inf
        for t in range(3):
            tok = int(toks[b, 4 + t])
            assert tok == O.sample_token(logits[t], 0.7, O.gumbel_from_bits(O.noise_bits(7, b, t, vocab)))[0]
            if np.isnan(value):
                assert np.isnan(lps[b, t])
            else:
                assert abs(lps[b, t] - O.log_softmax_at(logits[t], 0.7, tok)) <= 1e-4
            if tok == cfg.eos_id:
                break
