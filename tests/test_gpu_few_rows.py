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
    # head sizes without a decode kernel of their own: the general pass, with few-rows products or split ones
    "hd32": (256, 8, 32, 8, 512, 300), "hd96": (768, 8, 96, 24, 512, 300), "hd32-1024": (1024, 32, 32, 8, 1024, 300),
    "hd32-2112": (2112, 66, 32, 8, 256, 300), "hd32-4096": (4096, 128, 32, 8, 128, 300),
    # LM heads of more than 1024 blocks and 33 or 34 steps (bf16 / fp32): the form of eight waves
    "head2112": (2112, 33, 64, 16, 128, 32800), "head1088": (1088, 17, 64, 16, 128, 32800),
}

DECODES = [  # shape, sequences, shortest and longest query
    ("hd64", 1, 1, 1), ("hd80", 1, 300, 300), ("hd16", 15, 1, 40), ("hd256", 16, 5, 90), ("hd80", 17, 1, 70),
    ("hd128", 32, 3, 33), ("hd64", 33, 1, 130), ("hd80", 48, 60, 61), ("hd16", 49, 1, 9), ("hd64", 64, 1, 20),
    ("hd128", 64, 1, 8), ("hd64", 65, 1, 8), ("hd80", 128, 1, 40), ("hd256", 129, 1, 9), ("hd16", 193, 1, 70),
    ("hd80", 256, 1, 8), ("hd64", 257, 1, 8), ("hd32", 1, 1, 5), ("hd32", 64, 1, 9), ("hd96", 56, 3, 20), ("hd96", 57, 1, 9),
    ("hd32-1024", 32, 1, 9), ("hd32-1024", 33, 1, 9), ("hd32-1024", 64, 5, 40), ("hd32-2112", 3, 1, 9),
    ("hd32-4096", 4, 1, 9), ("hd32-4096", 5, 1, 9), ("head2112", 1, 1, 9), ("head2112", 8, 1, 9), ("head1088", 1, 1, 9),
    ("head1088", 8, 1, 9)
]
# One layer of the wide models, whose products take the other forms of the kernel (64 to 128 columns per block, K loops
# long enough to be pipelined): sequences at the edges of the row tiles, and several row tiles of the forms of 64 and 80
# columns up to the line to the other decode pass
WIDTHS = {"1b": (2048, 8, 256, 64, 8192), "2.8b": (2560, 32, 80, 20, 10240), "6.9b": (4096, 32, 128, 32, 16384)}
WIDE = [("1b", 1), ("1b", 17), ("1b", 48), ("1b", 64), ("2.8b", 16), ("2.8b", 32), ("2.8b", 48), ("2.8b", 64), ("6.9b", 5),
        ("6.9b", 31), ("6.9b", 37), ("6.9b", 64), ("2.8b", 65), ("2.8b", 128), ("1b", 129), ("1b", 192)]
WIDE_FP32 = [("1b", 1), ("1b", 17), ("1b", 33), ("1b", 64), ("2.8b", 1), ("2.8b", 64), ("6.9b", 64)]
MANY_FP32 = [("1b", 3, 50), ("1b", 4, 75)]  # rescoring: width, sequences, tokens of each


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("shape,B,lo,hi", DECODES)
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


@pytest.mark.parametrize("shape,B,few", [
    ("hd64", 1, True), ("hd64", 256, True), ("hd64", 257, False), ("hd32", 4, False),  # a size, a head size without a kernel
    ("d1536", 64, True), ("d1536", 192, True), ("d1536", 193, False),  # weights of a layer times row tiles up to 5 * 2^25
    ("d4160", 1, False)])  # a width the decode LayerNorm does not take
def test_which_decode_pass(shape, B, few):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_17031_amd as P
    more = {"d1536": (1536, 24, 64, 16, 11456, 64), "d4160": (4160, 65, 64, 16, 64, 64)}
    d, H, hd, r, F, V = SHAPES.get(shape) or more[shape]
    cfg = ModelConfig(1, d, H, hd, r, F, vocab=V, dtype="bf16", pad_id=V)
    p = P.Policy(cfg, make_weights(cfg, 77, variant="test"))
    p.profile_enable()
    p.rollout_generate(np.ones((B, 2), np.int32), np.ones((B, 2), np.uint8), 11, 0.7, 2)
    assert ("gemm_decode_qkv_fc1" in p.profile_read()) == few


@pytest.mark.parametrize("F,few", [(15104, True), (15168, False)])
def test_the_line_between_the_decode_passes(F, few):
    """129 sequences are three row tiles: weights of a layer times three, 167.5 and 168.1 M on either side of 5 * 2^25."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_17031_amd as P
    cfg = ModelConfig(1, 1536, 24, 64, 16, F, vocab=64, dtype="bf16", pad_id=64)
    p = P.Policy(cfg, make_weights(cfg, 77, variant="test"))
    p.profile_enable()
    p.rollout_generate(np.ones((129, 2), np.int32), np.ones((129, 2), np.uint8), 11, 0.7, 2)
    assert ("gemm_decode_qkv_fc1" in p.profile_read()) == few


@pytest.fixture(scope="module")
def wide_model():
    kept = {}

    def get(width, dtype):
        if (width, dtype) not in kept:
            kept.clear()  # one at a time: a layer at width 4096 is 1.6 GB in float64
            d, H, hd, r, F = WIDTHS[width]
            cfg = ModelConfig(1, d, H, hd, r, F, vocab=515, dtype=dtype, pad_id=515)
            w = make_weights(cfg, 78, variant="test")
            from oracle import neox_oracle as O
            kept[width, dtype] = (cfg, w, O.OracleModel(w, cfg))
        return kept[width, dtype]
    return get


@pytest.mark.parametrize("dtype,width,B", [("bf16", *c) for c in sorted(WIDE)] + [("fp32", *c) for c in sorted(WIDE_FP32)])
def test_decode_at_the_width_of_a_wide_model(wide_model, dtype, width, B):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_17031_amd as P
    from oracle import neox_oracle as O
    cfg, w, oracle = wide_model(width, dtype)
    g = np.random.default_rng(B)
    hi, N = 12, 4
    lens = g.integers(1, hi + 1, size=B)
    lens[-1] = hi
    mask = (np.arange(hi)[None, :] >= (hi - lens)[:, None]).astype(np.uint8)
    queries = np.where(mask == 1, g.integers(1, 515, size=(B, hi)), 515).astype(np.int32)
    toks, lps, _ = (x.cpu().numpy() for x in P.Policy(cfg, w).rollout_generate(queries, mask, 12, 0.7, N))
    for rep in O.verify_rollout(oracle, toks, mask, 12, 0.7, N, rows=sorted({0, B // 2, 64 if B > 64 else 0, B - 1})):
        assert rep["deficit"] <= (0.0 if dtype == "fp32" else NEAR_TIE), rep
        assert abs(lps[rep["row"], rep["step"]] - rep["logprob"]) <= TOL[dtype], rep


@pytest.mark.parametrize("width,B,L", MANY_FP32)
def test_fp32_rescoring_of_many_rows(wide_model, width, B, L):
    """The products of an fp32 pass over many rows are the few-rows kernel's too, its forms of up to 128 columns with
    several row tiles."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_17031_amd as P
    from oracle import neox_oracle as O
    cfg, w, oracle = wide_model(width, "fp32")
    g = np.random.default_rng(L)
    tokens, mask = g.integers(1, 515, size=(B, L)).astype(np.int32), np.ones((B, L), np.uint8)
    lp, val = (x.cpu().numpy() for x in P.Policy(cfg, w).score_sequences(tokens, mask, 0.7))
    olp, oval = O.score_sequences(oracle, tokens, mask, 0.7)
    assert np.abs(lp - olp).max() <= TOL["fp32"]
    assert np.abs(val - oval).max() <= TOL["fp32"] * max(1.0, float(np.abs(oval).max()))


def test_weights_at_any_float_address(monkeypatch):
    """An fp32 model whose arrays start four bytes past a 16-byte boundary: decode takes the general pass, whose kernels
    read them float by float, and the results stand."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_17031_amd as P
    from oracle import neox_oracle as O
    d, H, hd, r, F, V = SHAPES["hd64"]
    cfg = ModelConfig(2, d, H, hd, r, F, vocab=V, dtype="fp32", pad_id=V)
    w = make_weights(cfg, 77, variant="test")
    to = torch.Tensor.to

    def shifted(t, *args, **kw):
        t = to(t, *args, **kw)
        return torch.cat([t.new_zeros(1), t.flatten()])[1:].view(t.shape) if t.is_cuda else t

    g = np.random.default_rng(5)
    B, Lq, N = 3, 9, 5
    queries, mask = g.integers(1, V, size=(B, Lq)).astype(np.int32), np.ones((B, Lq), np.uint8)
    with monkeypatch.context() as m:
        m.setattr(torch.Tensor, "to", shifted)
        pol = P.Policy(cfg, w)
    assert all(t.data_ptr() % 16 == 4 for t in pol._dev.values())
    for p, few in ((pol, False), (P.Policy(cfg, w), True)):
        p.profile_enable()
        toks, lps, _ = (x.cpu().numpy() for x in p.rollout_generate(queries, mask, 11, 0.7, N))
        assert ("gemm_decode_qkv_fc1" in p.profile_read()) == few
        for rep in O.verify_rollout(O.OracleModel(w, cfg), toks, mask, 11, 0.7, N, rows=list(range(B))):
            assert rep["deficit"] <= 0.0 and abs(lps[rep["row"], rep["step"]] - rep["logprob"]) <= TOL["fp32"], rep


@pytest.mark.parametrize("B,d,hd", [(1, 128, 64), (17, 128, 64), (64, 128, 64), (65, 2048, 32), (256, 2048, 32)])
def test_gelu_of_negative_inputs(B, d, hd):
    """FC1 outputs in [-4, -3], where GELU is x * Phi(x) with Phi down to 3e-5: an absolute error that fp16 would hide
    at 1 is a few per cent there.  Hidden values depend on b_fc1 alone and are all the residual stream holds, so their
    relative error is the logits'.  Bound: fp16 rounding of the hidden values and of the final LayerNorm's output, each
    2^-10 / sqrt(12) of a value (rms, worst case), on logits / T of standard deviation S: 4e-4 S, times three.  A GELU
    that is 2.6e-5 off (the form the large products use) gives 5e-3 S.  Beyond 64 sequences the decode passes are the large
    kernel's, which takes the erf form at wide models; the first draw, the prefill's, is left out."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_17031_amd as P
    from oracle import neox_oracle as O
    from synth.inputs import round_to_bf16
    F, V, N = 512, 300, 8
    cfg = ModelConfig(1, d, d // hd, hd, hd // 4, F, vocab=V, dtype="bf16", pad_id=V)
    w = make_weights(cfg, 77, variant="test")
    g = np.random.default_rng(B)
    w["layers.0.w_o"][:], w["layers.0.b_o"][:], w["layers.0.w_fc1"][:], w["layers.0.b_fc2"][:] = 0, 0, 0, 0
    w["layers.0.b_fc1"] = round_to_bf16(g.uniform(-4, -3, F).astype(np.float32))
    w["layers.0.w_fc2"] = round_to_bf16(60 * g.standard_normal((d, F), dtype=np.float32))
    w["embed_out"] = round_to_bf16(np.float32(0.3 * (128 / d) ** 0.5) * g.standard_normal((V, d), dtype=np.float32))
    queries = g.integers(1, V, size=(B, 3)).astype(np.int32)
    mask = np.ones((B, 3), np.uint8)
    toks, lps, _ = (x.cpu().numpy() for x in P.Policy(cfg, w).rollout_generate(queries, mask, 3, 0.7, N))
    m = O.OracleModel(w, cfg)
    err, spread = [], []
    for b in range(B):
        x, _ = O.forward_sequence(m, toks[b], np.arange(3 + N))
        logits, _ = O.heads(m, x[2:-1])
        for t in range(N):
            if t == 0 and B > 64:
                continue
            err.append(lps[b, t] - O.log_softmax_at(logits[t], 0.7, int(toks[b, 3 + t])))
            spread.append(logits[t].std() / 0.7)
            if toks[b, 3 + t] == cfg.eos_id:
                break
    assert np.sqrt(np.mean(np.square(err))) <= 3 * 4e-4 * np.mean(spread)


@pytest.mark.parametrize("hd", [16, 64, 256])  # 1 / sqrt(hd) is exact: scores are, too
def test_fp32_softmax_weights(hd):
    """The fp32 decode attention's softmax weights, one by one: cached row j has the exact score -x_j (50 to 80 below the
    new row's) and a one in column j of V, so column j of the result is exp(-x_j) / (1 + sum).  Bound: two exponentials of
    1 ulp each (a wave's rescaling is one more) and five roundings, 2 * 2^-23 + 5 * 2^-24 = 5.4e-7.  exp(x) as the base-2
    instruction on a rounded x * log2(e) is up to 4.4e-6 off there."""
    import ctypes as C
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_17031_amd as P
    attn = P.load_library()["_ZN4rlhf23launch_attn_decode_ropeEiPKvPvS2_liPKiiiS4_iiiPKfS6_S2_iP12ihipStream_t"]
    vp, i32 = C.c_void_p, C.c_int
    attn.argtypes = [i32, vp, vp, vp, C.c_long, i32, vp, i32, i32, vp, i32, i32, i32, vp, vp, vp, i32, vp]
    n, extra = hd, 4
    g = np.random.default_rng(hd)
    score = -np.round(16 * g.uniform(50, 80, n)) / 16
    dev = lambda a, t=torch.float32: torch.as_tensor(a, dtype=t, device="cuda:0").contiguous()  # noqa: E731
    k, v = np.zeros((n + extra, hd)), np.zeros((n + extra, hd))
    k[:n, 0], v[:n] = score, np.eye(n)
    new = np.zeros((3, hd))  # q, k, v of the new row: score 0, value 0
    new[0, 0] = np.sqrt(hd)
    kc, vc, qkv = dev(k), dev(v), dev(new)
    out = torch.zeros(16, hd, device="cuda:0")  # packed: 16-byte chunks of 16 rows
    length, off = dev([n], torch.int32), dev([0], torch.int32)
    rc = attn(0, qkv.data_ptr(), kc.data_ptr(), vc.data_ptr(), extra, 1, length.data_ptr(), 0, n + 1, off.data_ptr(), 1, hd,
              0, None, None, out.data_ptr(), hd, torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    got = out.view(hd // 4, 16, 4)[:, 0].reshape(hd).cpu().numpy().astype(np.float64)
    want = np.exp(score) / (1 + np.exp(score).sum())
    assert np.abs(got / want - 1).max() <= 5.4e-7


def test_output_embedding_of_more_than_4_gib():
    """A vocabulary whose output embedding is larger than 4 GiB: the tokens at both ends of the table are told apart in
    the decode passes.  Only 256 rows at either end are not zero; a row offset cut to 32 bits would land on row
    v - 262144 for v >= 262144."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_17031_amd as P
    from oracle import neox_oracle as O
    d, V, ends = 4096, 262144 + 256, 256
    cfg = ModelConfig(1, d, 32, 128, 32, 64, vocab=V, dtype="fp32", pad_id=V)
    w = make_weights(cfg.with_(vocab=512), 5, variant="test")
    for name in ("embed_in", "embed_out"):
        small, w[name] = w[name], np.zeros((V, d), np.float32)  # (zero pages: only the ends are backed by memory)
        w[name][:ends], w[name][-ends:] = small[:ends], small[ends:]
    w["embed_out"][:ends] *= 8  # sampled tokens come from the ends: logits of N(0, 10)
    w["embed_out"][-ends:] *= 8
    g = np.random.default_rng(0)
    B, Lq, N = 2, 4, 6
    queries = g.integers(1, ends, size=(B, Lq)).astype(np.int32)
    mask = np.ones((B, Lq), np.uint8)
    pol = P.Policy(cfg, w)
    toks, lps, _ = (x.cpu().numpy() for x in pol.rollout_generate(queries, mask, 3, 0.7, N))
    pol.close()
    # the same model without the zero rows, whose logit is 0 and whose noise is at most 22.9
    keep = np.r_[0:ends, V - ends:V]
    m = O.OracleModel({**w, "embed_in": w["embed_in"][keep], "embed_out": w["embed_out"][keep]}, cfg.with_(vocab=2 * ends))
    for b in range(B):
        seq = np.concatenate([queries[b], toks[b, Lq:]])
        small = np.where(seq >= ends, seq - (V - 2 * ends), seq)
        assert ((seq < ends) | (seq >= V - ends)).all(), seq
        x, _ = O.forward_sequence(m, small, np.arange(seq.size))
        logits, _ = O.heads(m, x[Lq - 1:-1])
        for t in range(N):
            full = np.zeros(V)
            full[keep] = logits[t]
            score = O.sample_token(full, 0.7, O.gumbel_from_bits(O.noise_bits(3, b, t, V)))[2]
            assert int(np.argmax(score)) == toks[b, Lq + t], (b, t)
            assert abs(O.log_softmax_at(full, 0.7, int(toks[b, Lq + t])) - lps[b, t]) <= TOL["fp32"], (b, t)
    assert (toks[:, Lq + 1:] >= V - ends).any()  # decode passes did sample beyond the 32-bit range
