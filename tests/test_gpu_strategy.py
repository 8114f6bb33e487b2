"""Per-part strategy on the GPU (Sec. 4.2: each linear part runs in INT4 or in a higher-bit type; the
FFN pair may hand codes over in the epilogue): w4a4_part_linear and w4a4_ffn against the oracle and,
bit for bit, against the entry points they are built from; the tuner's result against its own timings."""
import numpy as np
import pytest
import torch

from tests.gpu_util import dev, f16_close, f16_steps, has_gpu, host

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not has_gpu(), reason="needs a GPU")]


@pytest.fixture(scope="module")
def B():
    from paper_2301_12017_amd import binding
    binding.lib()
    return binding


def _xw(seed, M, N, K):
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((M, K)).astype(np.float32).astype(np.float16)
    W = (rng.standard_normal((N, K)) * 0.02).astype(np.float16)
    b = (rng.standard_normal(N) * 0.01).astype(np.float16)
    return X, W, b


# one-kernel shape; operand-layout two-call shape with a ragged last tile; canonical two-call shape (K > 4096)
PART_SHAPES = [(48, 96, 128), (1100, 768, 256), (40, 64, 8192)]


@pytest.mark.parametrize("M,N,K", PART_SHAPES)
@pytest.mark.parametrize("act", [0, 1])
def test_part_linear_int4(B, orc, M, N, K, act):
    X, W, b = _xw(M + N + K, M, N, K)
    P = B.Part(dev(W), M, dev(b), act)
    got = B.part_linear(dev(X), P, True)
    # the calls it stands for, bit for bit
    A = B.quantize_act(dev(X), B.SYM, layout=P.w4.layout)
    ref = B.linear(A, P.w4, dev(b), act)
    assert torch.equal(got, ref)
    want = orc.part_linear(X, W, True, b, act)
    if act == 0:
        assert np.array_equal(host(got).view(np.uint16), want.view(np.uint16))
    else:
        ok, ratio = f16_close(host(got), want)
        assert ok, ratio


@pytest.mark.parametrize("K,M,N,one", [(768, 500, 1152, True), (768, 640, 1600, False), (512, 800, 1152, True), (640, 600, 1600, True),
                                       (640, 601, 1600, False), (576, 960, 544, True), (576, 960, 576, False), (960, 640, 832, False), (1152, 512, 1024, True), (1152, 512, 1056, False)])
def test_part_linear_in_one_launch_or_two(B, K, M, N, one):
    """Few tokens take one launch, which needs no workspace: up to 960 tiles of 32 x 32, 512 of more than 600 tokens where
    the kernel has K at run time."""
    g = torch.Generator(device="cuda").manual_seed(K + M)
    X = torch.randn((M, K), device="cuda", generator=g).half()
    P = B.Part((torch.randn((N, K), device="cuda", generator=g) * 0.02).half(), M, layout=0)
    ws = torch.full((M * K + (1 << 16),), 0xAB, dtype=torch.uint8, device="cuda")
    out = B.part_linear(X, P, True, workspace=ws)
    assert bool((ws == 0xAB).all()) == one
    A = B.quantize_act(X, 0)
    assert torch.equal(out.view(torch.int16), B.linear(A, P.w4).view(torch.int16))


@pytest.mark.parametrize("M,N,K", [(48, 96, 128), (1100, 768, 256), (40, 64, 4096)])
@pytest.mark.parametrize("act", [0, 1])
def test_part_linear_int8(B, orc, M, N, K, act):
    X, W, b = _xw(M + N + K + 1, M, N, K)
    P = B.Part(dev(W), M, dev(b), act)
    got = B.part_linear(dev(X), P, False)
    want = orc.part_linear(X, W, False, b, act)
    if act == 0:
        assert np.array_equal(host(got).view(np.uint16), want.view(np.uint16))
    else:
        ok, ratio = f16_close(host(got), want)
        assert ok, ratio


def test_part_linear_asymmetric_grouped(B, orc):
    M, N, K = 70, 64, 256
    X, W, b = _xw(9, M, N, K)
    X = (X.astype(np.float32) + 0.7).astype(np.float16)
    P = B.Part(dev(W), M, dev(b), 0, mode=B.ASYM, group=128)
    got = B.part_linear(dev(X), P, True)
    want = orc.part_linear(X, W, True, b, 0, mode=orc.ASYM, group=128)
    ok, ratio = f16_close(host(got), want)
    assert ok, ratio


def test_part_linear_reads_a_column_slice_and_reuses_a_workspace(B, orc):
    M, N, K = 36, 64, 128
    X, W, b = _xw(4, M, N, 2 * K)
    Xd = dev(X)
    P = B.Part(dev(W[:, :K].copy()), M, dev(b), 0)
    ws = torch.empty(1 << 16, dtype=torch.uint8, device="cuda")
    for int4 in (True, False, True):
        got = B.part_linear(Xd[:, K:], P, int4, workspace=ws)
        want = orc.part_linear(np.ascontiguousarray(X[:, K:]), W[:, :K].copy(), int4, b, 0)
        assert np.array_equal(host(got).view(np.uint16), want.view(np.uint16))


# (M, h, ffn): one-kernel parts; a mix (FFN1 in the operand layout, FFN2 one-kernel); both in the operand layout
FFN_SHAPES = [(40, 128, 256), (1100, 256, 1024), (2100, 512, 1024)]


def _ffn_inputs(seed, M, h, f):
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((M, h)).astype(np.float32).astype(np.float16)
    W1 = (rng.standard_normal((f, h)) * 0.05).astype(np.float16)
    W2 = (rng.standard_normal((h, f)) * 0.05).astype(np.float16)
    b1 = (rng.standard_normal(f) * 0.02).astype(np.float16)
    b2 = (rng.standard_normal(h) * 0.02).astype(np.float16)
    return X, W1, b1, W2, b2


def _pair_equal(got, want, exact):
    if exact:
        assert np.array_equal(got.view(np.uint16), want.view(np.uint16))
        return
    # a differing intermediate moves a 4-bit code of the second part now and then, which shifts that token's outputs
    # by a fraction of the quantization noise: most values identical, the rest bounded in the mean
    same, _ = f16_steps(got, want)
    g, w = got.astype(np.float64), want.astype(np.float64)
    assert same >= 0.99 and np.sqrt(np.mean((g - w) ** 2)) <= 5e-3 * np.sqrt(np.mean(w ** 2)), same


@pytest.mark.parametrize("M,h,f", FFN_SHAPES)
@pytest.mark.parametrize("strategy", [0, 4, 8, 12, 28])
def test_ffn_without_activation_matches_the_oracle(B, orc, M, h, f, strategy):
    """Without GELU every intermediate value is bit-identical on both sides on the canonical kernels, so the whole
    pair is.  From 1536 tokens up the INT4 parts run on the persistent operand-layout kernel, whose fp16 stores agree
    with the definition except on near-ties of the fp16 grid (one step): a stored intermediate that differs can
    move a code of FFN2's input, so the pair is then held to the tolerance and to 99 % identical values."""
    X, W1, b1, W2, b2 = _ffn_inputs(M + strategy, M, h, f)
    P1, P2 = B.Part(dev(W1), M, dev(b1), 0), B.Part(dev(W2), M, dev(b2), 0)
    got = host(B.ffn(dev(X), P1, P2, strategy))
    want = orc.ffn(X, W1, b1, 0, W2, b2, strategy)
    _pair_equal(got, want, exact=not (M >= 1536 and strategy & 12))


@pytest.mark.parametrize("M,h,f", FFN_SHAPES)
@pytest.mark.parametrize("strategy", [0, 4, 8, 12, 28])
def test_ffn_with_gelu_equals_its_building_blocks(B, orc, M, h, f, strategy):
    X, W1, b1, W2, b2 = _ffn_inputs(M + strategy + 50, M, h, f)
    P1, P2 = B.Part(dev(W1), M, dev(b1), 1), B.Part(dev(W2), M, dev(b2), 0)
    Xd = dev(X)
    got = B.ffn(Xd, P1, P2, strategy)
    if strategy & B.STRATEGY_FUSED_FFN:
        A = B.quantize_act(Xd, B.SYM, layout=P1.w4.layout)
        H = B.linear(A, P1.w4, dev(b1), 1, requant=True, requant_layout=P2.w4.layout)
        ref = B.linear(H, P2.w4, dev(b2), 0)
    else:
        H = B.part_linear(Xd, P1, bool(strategy & 4))
        ref = B.part_linear(H, P2, bool(strategy & 8))
    assert torch.equal(got, ref)
    # and the oracle's pair: a GELU value that differs in its last bit can move a code of the
    # intermediate by one step, so this comparison is statistical
    want = orc.ffn(X, W1, b1, 1, W2, b2, strategy).astype(np.float64)
    err = host(got).astype(np.float64) - want
    assert np.sqrt((err ** 2).mean()) < 5e-3 * np.sqrt((want ** 2).mean())


def test_ffn_is_repeatable_on_one_workspace(B):
    M, h, f = 1100, 256, 1024
    X, W1, b1, W2, b2 = _ffn_inputs(1, M, h, f)
    P1, P2 = B.Part(dev(W1), M, dev(b1), 1), B.Part(dev(W2), M, dev(b2), 0)
    Xd = dev(X)
    ws = torch.empty(32 << 20, dtype=torch.uint8, device="cuda")
    first = {s: B.ffn(Xd, P1, P2, s, workspace=ws).clone() for s in (28, 12, 0)}
    for s in (0, 28, 12, 28):
        assert torch.equal(B.ffn(Xd, P1, P2, s, workspace=ws), first[s])


def test_tuner_picks_what_its_timings_say(B, orc):
    for M, h, f in [(128, 768, 3072), (2048, 768, 3072)]:
        pick, part_us, fused_us = B.strategy_tune(M, h, f, iters=10)
        assert all(t > 0 for row in part_us for t in row) and fused_us > 0
        # the tuner's documented rule: timings within 3 % of each other count as equal
        snapped = [[min(a, b), min(a, b)] if abs(a - b) <= 0.03 * min(a, b) else [a, b] for a, b in part_us]
        unfused = snapped[2][1] + snapped[3][1]
        fused = unfused if 0 < fused_us - unfused <= 0.03 * unfused else fused_us
        assert pick == orc.pick_strategy(snapped, fused)
        assert B.strategy_lookup(M, h, f) == pick                      # remembered for this device
    assert B.strategy_lookup(136, 768, 3072) == 15                     # untuned shape: the built-in table


@pytest.mark.parametrize("M,h,f", [(12288, 768, 2048), (8200, 1024, 4096)])
def test_tuner_where_the_layer_takes_the_fp6_layout(B, orc, M, h, f):
    """Its synthetic INT4 weights are in that layout, too: sizes of their own, every option runs, the pick is remembered."""
    assert B.lib().w4a4_encoder_layer_prefers_fp6(M, h, f) == 1
    pick, part_us, fused_us = B.strategy_tune(M, h, f, iters=3)
    assert all(0 < t < 1e5 for row in part_us for t in row) and 0 < fused_us < 1e5
    assert B.strategy_lookup(M, h, f) == pick and B.fused_fault_check() is False


def _big(seed, M, h, f):
    """Full-size operands made on the device (the host copy of the weights and of the sampled rows goes to the oracle)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    rn = lambda *s, std=1.0: (torch.randn(s, device="cuda", generator=g) * std).half()
    return rn(M, h), rn(f, h, std=0.03), rn(f, std=0.02), rn(h, f, std=0.03), rn(h, std=0.02)


@pytest.mark.parametrize("int4", [True, False])
def test_part_linear_at_full_size_on_sampled_rows(B, orc, int4):
    """BERT-large MLP output at the bench's token count (12288 x 1024 x 4096): the GPU runs the whole part, the
    oracle the sampled token rows (rows are independent end to end)."""
    M, h, f = 12288, 1024, 4096
    X, W1, b1, W2, b2 = _big(3, M, f, h)                    # here: X [M, 4096], W1 [1024, 4096]
    P = B.Part(W1, M, b1, 0)
    got = B.part_linear(X, P, int4)
    rows = np.sort(np.concatenate([[0, M - 1], np.random.default_rng(1).choice(M, 6, replace=False)]))
    rt = torch.from_numpy(rows).cuda()
    want = orc.part_linear(host(X[rt]), host(W1), int4, host(b1), 0)
    _pair_equal(host(got[rt]), want, exact=not int4)               # INT4 at this size: the operand-layout kernel


@pytest.mark.parametrize("strategy", [12, 28])
def test_ffn_at_full_size_on_sampled_rows(B, orc, strategy):
    """The BERT-large FFN pair at 12288 tokens without an activation in between (so that both sides agree up to
    near-ties of the fp16 stores): separate quantize of the fp16 intermediate, and codes handed over in the epilogue."""
    M, h, f = 12288, 1024, 4096
    X, W1, b1, W2, b2 = _big(4, M, h, f)
    P1, P2 = B.Part(W1, M, b1, 0), B.Part(W2, M, b2, 0)
    assert P1.w4.layout == 1 and P2.w4.layout == 1           # the operand layout at this size
    got = B.ffn(X, P1, P2, strategy)
    rows = np.sort(np.concatenate([[0, M - 1], np.random.default_rng(2).choice(M, 4, replace=False)]))
    rt = torch.from_numpy(rows).cuda()
    want = orc.ffn(host(X[rt]), host(W1), host(b1), 0, host(W2), host(b2), strategy)
    _pair_equal(host(got[rt]), want, exact=False)


def test_parts_in_the_fp6_layout(B, orc):
    """Weights in the FP6 operand layout through the per-part calls: a part equals quantize_act + w4a4_linear bit for bit
    and the oracle's part; the fused FFN pair (FFN1 requantizes into FFN2's FP6 operand in its epilogue) equals the oracle's
    fused pair bit for bit without GELU; a pair with only one side in the layout is refused; so is the whole layer."""
    M, h, f = 700, 512, 1024
    X, W1, b1, W2, b2 = _ffn_inputs(21, M, h, f)
    P1 = B.Part(dev(W1), M, dev(b1), 0, layout=B.LAYOUT_FP6)
    P2 = B.Part(dev(W2), M, dev(b2), 0, layout=B.LAYOUT_FP6)
    got = B.part_linear(dev(X), P1, True)
    A = B.quantize_act(dev(X), B.SYM, layout=B.LAYOUT_FP6)
    assert torch.equal(got, B.linear(A, P1.w4, dev(b1), 0))
    assert np.array_equal(host(got).view(np.uint16), orc.part_linear(X, W1, True, b1, 0).view(np.uint16))
    pair = host(B.ffn(dev(X), P1, P2, 12))                      # both parts in INT4, an fp16 tensor between them
    assert np.array_equal(pair.view(np.uint16), orc.ffn(X, W1, b1, 0, W2, b2, 12).view(np.uint16))
    fused = host(B.ffn(dev(X), P1, P2, 28))                     # the codes handed over in FFN1's epilogue
    assert np.array_equal(fused.view(np.uint16), orc.ffn(X, W1, b1, 0, W2, b2, 28).view(np.uint16))
    assert B.fused_fault_check() is False
    Pm = B.Part(dev(W2), M, dev(b2), 0, layout=B.LAYOUT_MFMA)
    with pytest.raises(RuntimeError):
        B.ffn(dev(X), P1, Pm, 28)
