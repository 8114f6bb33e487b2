"""The FP16 attention stand-in and the whole encoder layer (Sec. 4.2: FP16 attention between the quantized
linears, LayerNorm after the attention output and the MLP, the launch sequence replayed from a graph for small
inputs): against the oracle, against the entry points the layer is composed of, and under graph replay."""
import numpy as np
import pytest
import torch

from tests.gpu_util import dev, has_gpu, host

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not has_gpu(), reason="needs a GPU")]


@pytest.fixture(scope="module")
def B():
    from paper_2301_12017_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("batch,seq,heads", [(1, 128, 12), (3, 37, 2), (2, 512, 1), (5, 1, 3), (1, 70, 16)])
def test_attention_against_the_oracle(B, orc, batch, seq, heads):
    rng = np.random.default_rng(batch + seq + heads)
    QKV = (rng.standard_normal((batch * seq, 3 * heads * 64)) * 1.5).astype(np.float16)
    got = host(B.attention(dev(QKV), batch, seq, heads)).astype(np.float64)
    want = orc.attention(QKV, batch, seq, heads)
    # fp32 sums of <= 512 terms and one fp16 rounding of the result
    assert np.abs(got - want).max() <= 1e-3 * np.abs(want) .max() + 1e-3 * np.sqrt((want ** 2).mean())
    np.testing.assert_allclose(got, want, rtol=2e-3, atol=2e-3 * np.sqrt((want ** 2).mean()))


@pytest.mark.parametrize("batch,heads", [(1, 3), (17, 12)])     # waves share a block of queries (above 32 tokens); a wave per block
@pytest.mark.parametrize("seq", [1, 31, 32, 33, 64, 65, 127, 128, 129, 255, 257, 511, 512])
def test_attention_at_the_edges_of_its_tiles(B, orc, batch, heads, seq):
    rng = np.random.default_rng(seq)
    QKV = (rng.standard_normal((batch * seq, 3 * heads * 64)) * 1.5).astype(np.float16)
    got = host(B.attention(dev(QKV), batch, seq, heads)).reshape(batch, seq, heads, 64).astype(np.float64)
    last = batch - 1                                             # the first and the last (sequence, head) of the launch
    for b, h in ((0, 0), (last, heads - 1)):
        one = np.ascontiguousarray(QKV.reshape(batch, seq, 3, heads, 64)[b, :, :, h]).reshape(seq, 192)
        want = orc.attention(one, 1, seq, 1)
        # one rounding to fp16; sums of `seq` fp32 terms (2^-24 each) of at most max|v|
        bound = 2.0 ** -11 * np.abs(want) + (seq + 64) * 2.0 ** -24 * np.abs(one[:, 128:].astype(np.float64)).max()
        assert np.all(np.abs(got[b, :, h] - want) <= bound)


@pytest.mark.parametrize("batch,heads", [(1, 3), (17, 12)])
def test_attention_with_infinite_keys_and_values(B, batch, heads):
    """Keys at -inf score (weight 0, a whole block of them first), an infinite value, a NaN: finite, infinite and NaN where
    the definition is."""
    seq, rng = 150, np.random.default_rng(8)
    x = rng.standard_normal((batch, seq, 3, heads, 64)).astype(np.float16)
    x[:, :, 0] = np.abs(x[:, :, 0]) + np.float16(0.01)            # queries > 0: a key of -inf scores -inf
    x[0, :40, 1, 0, 5] = -np.inf
    x[0, 60, 2, 1, 7] = np.inf
    x[0, 61, 2, 1, 8] = -np.inf
    x[0, 70, 2, 2, 9] = np.nan
    got = host(B.attention(dev(x.reshape(batch * seq, -1)), batch, seq, heads)).reshape(batch, seq, heads, 64)
    for head in range(3):
        q, k, v = (x[0, :, i, head].astype(np.float64) for i in range(3))
        s = q @ k.T / 8
        p = np.exp(s - s.max(axis=1, keepdims=True))
        want = (p[:, :, None] * v).sum(axis=1) / p.sum(axis=1, keepdims=True)
        # one rounding to fp16; 150 fp32 terms of at most max|v| each (2^-24)
        bound = 2.0 ** -11 * np.abs(want) + (seq + 64) * 2.0 ** -24 * np.abs(v[np.isfinite(v)]).max()
        with np.errstate(invalid="ignore"):
            near = np.isfinite(want) & (np.abs(got[0, :, head] - want) <= bound)
        assert np.all(near | (got[0, :, head] == want) | (np.isnan(want) & np.isnan(got[0, :, head])))


@pytest.mark.parametrize("batch,heads", [(1, 3), (17, 12)])     # waves share a block of queries (above 32 tokens); a wave per block
@pytest.mark.parametrize("order", ["up", "down", "mixed"])
@pytest.mark.parametrize("query,key", [(100, 1000), (3000, 5000), (4400, 5000), (4700, 5000), (-4700, 5000), (10000, 10000), (12000, 12000),
                                       (16000, 16000), (20000, 20000), (-20000, 20000), (60000, 60000)])
def test_attention_of_large_finite_scores(B, batch, heads, query, key, order):
    """q.k = query * key + step * j, exact in FP32, up to 3.6e9 (and below zero): softmax of the differences, although the scores
    times a constant are not exact (from 2.3e7 on a rounded one is off by a quarter and more, by 32 at 3e9).  Neighbouring
    queries differ in sign and by 1024."""
    seq, rng = 150, np.random.default_rng(abs(query) + key)
    step = max(8, int(2 * np.spacing(np.float32(abs(query) * key))))
    j = rng.integers(0, 6, seq)
    j = {"up": np.sort(j), "down": np.sort(j)[::-1], "mixed": j}[order]
    x = rng.standard_normal((batch, seq, 3, heads, 64)).astype(np.float16)
    x[:, :, :2] = 0
    x[:, :, 0, :, 5], x[:, :, 1, :, 5] = (query * np.array([1, 2.0 ** -10, -1, -2.0 ** -10]))[np.arange(seq) % 4][:, None], key
    x[:, :, 0, :, 60], x[:, :, 1, :, 60] = step, j[None, :, None]
    x[0, 40:, 1, 0, 5] = -key / 2                                 # one head whose scores cross zero, and the limit
    got = host(B.attention(dev(x.reshape(batch * seq, -1)), batch, seq, heads)).reshape(batch, seq, heads, 64).astype(np.float64)
    for b, h in ((0, 0), (0, 1), (batch - 1, heads - 1)):
        q, k, v = (x[b, :, i, h].astype(np.float64) for i in range(3))
        s = q @ k.T / 8
        p = np.exp(s - s.max(axis=1, keepdims=True))
        want = p @ v / p.sum(axis=1, keepdims=True)
        # one rounding to fp16; exponents of at most 5 * step / 8 to one part in 2^23, `seq` terms of at most max|v|
        bound = 2.0 ** -11 * np.abs(want) + (seq + 64) * 2.0 ** -24 * np.abs(v).max()
        assert np.all(np.abs(got[b, :, h] - want) <= bound), np.max(np.abs(got[b, :, h] - want))


@pytest.mark.parametrize("batch,heads", [(1, 3), (17, 12)])     # waves share a block of queries (above 32 tokens); a wave per block
@pytest.mark.parametrize("depth", [2, 6, 9, 11, 14, 17])
@pytest.mark.parametrize("where", [0, 70, 149])
def test_attention_of_small_weights(B, batch, heads, depth, where):
    """The largest weight of a row meets a value of zero, so that the result consists of weights around e^-depth alone."""
    seq, rng = 150, np.random.default_rng(depth)
    x = rng.standard_normal((batch, seq, 3, heads, 64)).astype(np.float16)
    x[:, :, :2] = 0
    x[:, :, 0, :, 5], x[:, :, 1, :, 5] = 8, np.float16(rng.uniform(-0.5, 0.5, seq))[None, :, None]
    x[:, :, 2] = rng.uniform(0.5, 1, (batch, seq, heads, 64)) * min(60000, 2.0 ** -10 * np.exp(depth))
    x[:, where, 1, :, 5], x[:, where, 2] = depth, 0
    got = host(B.attention(dev(x.reshape(batch * seq, -1)), batch, seq, heads)).reshape(batch, seq, heads, 64).astype(np.float64)
    for b, h in ((0, 0), (batch - 1, heads - 1)):
        q, k, v = (x[b, :, i, h].astype(np.float64) for i in range(3))
        s = q @ k.T / 8
        p = np.exp(s - s.max(axis=1, keepdims=True))
        want = p @ v / p.sum(axis=1, keepdims=True)
        assert np.all(want > 2.0 ** -14)
        # relative: one rounding to fp16; weights of at least e^-(depth + 0.5) to 2^-41 (2^-15.8 of them at depth 17, their sum to less)
        # and, with exponents of at most 25 to one part in 2^24, to 2^-19
        assert np.all(np.abs(got[b, :, h] - want) <= want * (2.0 ** -11 + 2.0 ** -15))


@pytest.mark.parametrize("batch,heads,seq", [(1, 3, 150), (1, 2, 20), (17, 12, 150), (60, 12, 40)])
def test_attention_with_infinite_values_of_small_weight(B, batch, heads, seq):
    """Infinite values count where their weight is far below an FP16 number (e^-30) but not zero in FP32, make a NaN where it is
    (e^-120) or where both signs meet, and touch no other feature; rows of keys that all score -inf are NaN."""
    rng = np.random.default_rng(seq)
    x = rng.standard_normal((batch, seq, 3, heads, 64)).astype(np.float16)
    b, h = batch - 1, heads - 1                                   # the last (sequence, head) of the launch, and its neighbour's first
    x[b, :, 0, h] = 1.0
    x[b, :, 1, h] = 0.0
    x[b, 11, 1, h, :40] = -6.0                                    # scores 0, and -30 and -120 at two keys
    x[b, seq - 1, 1, h, :] = -15.0
    x[b, 11, 2, h, 5], x[b, 11, 2, h, 40] = np.inf, -np.inf
    x[b, 3, 2, h, 40], x[b, 3, 2, h, 41] = np.inf, -np.inf
    x[b, seq - 1, 2, h, 63] = np.inf
    x[b, 0, 2, h, 17] = np.nan
    x[0, :, 0, 0] = 1.0
    x[0, :, 1, 0, 0] = -np.inf
    got = host(B.attention(dev(x.reshape(batch * seq, -1)), batch, seq, heads)).reshape(batch, seq, heads, 64).astype(np.float64)
    one = got[b, :, h]
    assert np.all(one[:, 5] == np.inf) and np.all(one[:, 41] == -np.inf)
    assert np.all(np.isnan(one[:, [17, 40, 63]]))
    assert np.all(np.isfinite(np.delete(one, [5, 17, 40, 41, 63], axis=1)))
    assert np.all(np.isnan(got[0, :, 0]))
    assert np.all(np.isfinite(got[0, :, 1:-1])) and np.all(np.isfinite(got[1:-1]))


def test_attention_costs_no_more_with_nan_or_infinity(B):
    """A NaN key, a NaN value or an infinite value in every head: a scan of the values and one key scored again at most (1.0,
    1.15 and 1.2 times the clean 33 us), not every score of every row by every lane (160 to 1700 times)."""
    batch, seq, heads = 16, 512, 12
    clean = np.random.default_rng(4).standard_normal((batch, seq, 3, heads, 64)).astype(np.float16)

    def us(x):
        q = dev(x.reshape(batch * seq, -1))
        best = np.inf
        for _ in range(8):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            for _ in range(5):
                B.attention(q, batch, seq, heads)
            e[1].record()
            e[1].synchronize()
            best = min(best, e[0].elapsed_time(e[1]) * 200)
        return best

    base = us(clean)
    for part, value in ((1, np.nan), (2, np.nan), (2, np.inf)):
        x = clean.copy()
        x[:, 100, part, :, 9] = value
        assert us(x) < 4 * base, (part, value)


def test_attention_of_peaked_scores_does_not_overflow(B, orc):
    batch, seq, heads = 1, 64, 2
    rng = np.random.default_rng(3)
    QKV = (rng.standard_normal((seq, 3 * heads * 64)) * 12).astype(np.float16)      # scores of a few hundred
    got = host(B.attention(dev(QKV), batch, seq, heads)).astype(np.float64)
    want = orc.attention(QKV, batch, seq, heads)
    assert np.isfinite(got).all()
    np.testing.assert_allclose(got, want, rtol=3e-3, atol=3e-2)


def _layer(B, seed, batch, seq, heads, h, f, layout=None):
    rng = np.random.default_rng(seed)
    n = lambda *s, std=1.0: (rng.standard_normal(s) * std).astype(np.float16)
    t = dict(X=n(batch * seq, h), Wqkv=n(3 * h, h, std=0.05), bqkv=n(3 * h, std=0.02), Wao=n(h, h, std=0.05),
             bao=n(h, std=0.02), W1=n(f, h, std=0.05), b1=n(f, std=0.02), W2=n(h, f, std=0.05), b2=n(h, std=0.02),
             g1=(1 + 0.1 * rng.standard_normal(h)).astype(np.float16), be1=n(h, std=0.1),
             g2=(1 + 0.1 * rng.standard_normal(h)).astype(np.float16), be2=n(h, std=0.1))
    d = {k: dev(v) for k, v in t.items()}
    L = B.EncoderLayer(batch, seq, heads, d["Wqkv"], d["bqkv"], d["Wao"], d["bao"], d["W1"], d["b1"], d["W2"], d["b2"],
                       d["g1"], d["be1"], d["g2"], d["be2"], 1e-12, layout=layout)
    return t, d, L


def _blocks(B, L, d, strategy):
    """The layer spelled out with the entry points it is made of."""
    X = d["X"]
    M, h = X.shape
    qkv = B.part_linear(X, L.qkv, bool(strategy & 1))
    ctx = B.attention(qkv, L.batch, L.seq, L.heads)
    ao = B.part_linear(ctx, L.attn_out, bool(strategy & 2))
    a1 = B._new_qact(M, h, B.SYM, 0, L.ffn1.w4.layout, X.device)
    x1 = torch.empty_like(X)
    B.layernorm_quantize(ao, X, d["g1"], d["be1"], 1e-12, out=a1, y=x1, layout=L.ffn1.w4.layout)
    if strategy & B.STRATEGY_FUSED_LN:
        if strategy & B.STRATEGY_FUSED_FFN:
            H = B.linear(a1, L.ffn1.w4, d["b1"], B.ACT_GELU, requant=True, requant_layout=L.ffn2.w4.layout)
            h2 = B.linear(H, L.ffn2.w4, d["b2"])
        else:
            H = B.linear(a1, L.ffn1.w4, d["b1"], B.ACT_GELU)
            h2 = B.part_linear(H, L.ffn2, bool(strategy & 8))
    else:
        h2 = B.ffn(x1, L.ffn1, L.ffn2, strategy & 31)
    a2 = B._new_qact(M, h, B.SYM, 0, 0, X.device)
    out = torch.empty_like(X)
    B.layernorm_quantize(h2, x1, d["g2"], d["be2"], 1e-12, out=a2, y=out)
    return out


STRATEGIES = [0, 4, 15, 15 | 32, 31, 31 | 32, 7 | 32]


@pytest.mark.parametrize("shape", [(1, 128, 12, 768, 3072), (16, 128, 4, 256, 1024), (3, 21, 2, 128, 256)])
@pytest.mark.parametrize("strategy", STRATEGIES)
def test_layer_equals_its_building_blocks(B, shape, strategy):
    batch, seq, heads, h, f = shape
    t, d, L = _layer(B, sum(shape), batch, seq, heads, h, f)
    got = L(d["X"], strategy)
    assert torch.equal(got, _blocks(B, L, d, strategy))
    assert torch.isfinite(got.float()).all()


@pytest.mark.parametrize("strategy", STRATEGIES)
def test_layer_against_the_oracle(B, orc, strategy):
    batch, seq, heads, h, f = 2, 24, 2, 128, 256
    t, d, L = _layer(B, 77, batch, seq, heads, h, f)
    got = host(L(d["X"], strategy)).astype(np.float64)
    want = orc.encoder_layer(t["X"], batch, seq, heads, t["Wqkv"], t["bqkv"], t["Wao"], t["bao"], t["W1"], t["b1"], t["W2"],
                             t["b2"], t["g1"], t["be1"], t["g2"], t["be2"], 1e-12, strategy).astype(np.float64)
    # last-bit differences of the attention / GELU / LayerNorm values move a few INT4 codes of the next part
    # by one step, so whole-layer agreement is statistical; the pieces are checked one by one elsewhere
    rms = np.sqrt((want ** 2).mean())
    assert np.sqrt(((got - want) ** 2).mean()) < 1e-2 * rms
    assert np.abs(got - want).max() < 0.25 * rms


def test_layer_replays_from_a_graph(B):
    """The b1/s128 BERT-base layer captured once and replayed: every replay equals the eager result, with
    eager work of the same library (which shares no buffer with the graph) in between."""
    batch, seq, heads, h, f = 1, 128, 12, 768, 3072
    t, d, L = _layer(B, 5, batch, seq, heads, h, f)
    _, d2, L2 = _layer(B, 6, batch, seq, heads, h, f)
    for strategy in (15, 31 | 32):
        eager = L(d["X"], strategy).clone()
        out = torch.empty_like(eager)
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            L(d["X"], strategy, out=out, stream=side.cuda_stream)              # warm-up on the capture stream
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            L(d["X"], strategy, out=out, stream=side.cuda_stream)
        for rep in range(4):
            out.zero_()
            other = L2(d2["X"], strategy)                                        # eager work between replays
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, eager), (strategy, rep)
            assert torch.isfinite(other.float()).all()


@pytest.mark.parametrize("shape", [(1, 128, 12, 768, 3072), (5, 100, 8, 512, 1024)])
@pytest.mark.parametrize("strategy", STRATEGIES)
def test_layer_with_weights_in_the_fp6_layout(B, shape, strategy):
    """Every INT4 part on the FP6 matrix instruction (LayerNorm writes the FP6 operand, the fused FFN pair hands FP6 codes
    over): the layer equals the entry points it is made of, and - the FP6 kernels and the canonical-layout kernels both
    follow the definition's operation order - the same layer with canonical weights, bit for bit."""
    batch, seq, heads, h, f = shape
    t, d, L6 = _layer(B, sum(shape), batch, seq, heads, h, f, layout=B.LAYOUT_FP6)
    got = L6(d["X"], strategy)
    assert torch.equal(got, _blocks(B, L6, d, strategy))
    _, _, L0 = _layer(B, sum(shape), batch, seq, heads, h, f, layout=B.LAYOUT_CANONICAL)
    assert torch.equal(got, L0(d["X"], strategy))
    assert B.fused_fault_check() is False


@pytest.mark.parametrize("shape,fp6", [((64, 128, 16, 1024, 4096), True), ((63, 130, 16, 1024, 4096), False),
                                       ((24, 512, 12, 768, 3072), True), ((96, 127, 12, 768, 3072), False),
                                       ((64, 192, 6, 384, 1536), False)])
def test_layer_takes_the_fp6_layout_from_many_tokens_on(B, shape, fp6):
    """From 8192 tokens at hidden size 1024, 12288 below it, the default layout of a layer is FP6 where every part can take it
    (384 features cannot: the GEMM wants 512); the outputs are those of the layer asked for in the canonical layout, whose
    kernels follow the same operation order, bit for bit, in every strategy."""
    batch, seq, heads, h, f = shape
    t, d, L = _layer(B, 1, batch, seq, heads, h, f)
    assert [p.w4.layout == B.LAYOUT_FP6 for p in (L.qkv, L.attn_out, L.ffn1, L.ffn2)] == [fp6] * 4
    if fp6:
        _, _, L0 = _layer(B, 1, batch, seq, heads, h, f, layout=B.LAYOUT_CANONICAL)
        for strategy in (15, 31, 31 | 32, 7):
            assert torch.equal(L(d["X"], strategy), L0(d["X"], strategy)), strategy
    assert B.fused_fault_check() is False


def test_fp6_layout_is_named_where_the_layer_is_faster_in_it(B):
    """Not for 512 features, nor past 3072 (up to 10 % slower there)."""
    fp6 = lambda M, h, f: B.lib().w4a4_encoder_layer_prefers_fp6(M, h, f)
    assert [fp6(M, 512, 2048) for M in (12288, 16384, 32768)] == [0, 0, 0]
    assert [fp6(M, 4096, 8192) for M in (8192, 12288, 32768)] == [0, 0, 0]
    assert [fp6(M, 3072, 6144) for M in (8191, 8192, 32768)] == [0, 1, 1]
    assert [fp6(M, 768, 3072) for M in (12287, 12288, 32768)] == [0, 1, 1]


@pytest.mark.parametrize("shape", [(1, 17, 8, 512, 2048), (1, 3, 16, 1024, 256), (1, 45, 12, 768, 3072), (3, 15, 8, 512, 3072),
                                   (5, 31, 12, 768, 3072), (2, 50, 16, 1024, 4096), (1, 31, 16, 1024, 4096)])
def test_layernorm_inside_ffn1(B, shape):
    """Few tokens: LayerNorm 1 is formed inside FFN1's kernel, in tiles of 16 x 32, 32 x 32 and 32 x 64, with ragged tokens: the
    layer equals the entry points it is made of (a LayerNorm launch of its own) bit for bit."""
    batch, seq, heads, h, f = shape
    for seed, strategy in ((1, 15), (2, 7)):
        t, d, L = _layer(B, seed, batch, seq, heads, h, f)
        assert torch.equal(L(d["X"], strategy), _blocks(B, L, d, strategy))


def test_layernorm_inside_ffn1_takes_and_refuses_what_the_parts_do(B):
    """Infinities, NaN and sums past fp16's range give what the launches one by one give; a weight group that is no divisor of K
    is refused by that path as by every other."""
    batch, seq, heads, h, f = 1, 45, 12, 768, 3072
    t, d, L = _layer(B, 3, batch, seq, heads, h, f)
    for i, v in enumerate((np.inf, -np.inf, np.nan, 65504.0)):
        d["X"][7 * i + 2, 5 + 100 * i] = float(v)
        d["X"][7 * i + 3, 5 + 100 * i: 9 + 100 * i] = float(v)
    d["be1"][9], d["g1"][600] = 60000.0, 60000.0
    got, want = L(d["X"], 15), _blocks(B, L, d, 15)
    assert torch.equal(torch.isnan(got), torch.isnan(want)) and torch.isnan(got).any()
    assert torch.equal(torch.nan_to_num(got, nan=1.0).view(torch.int16), torch.nan_to_num(want, nan=1.0).view(torch.int16))
    L.c.ffn1.w4.group = 2 * h
    L.workspace = torch.empty((1 << 26,), dtype=torch.uint8, device="cuda")
    with pytest.raises(B.W4A4Error):
        L(d["X"], 15)
