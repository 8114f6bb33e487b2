"""w4a4_linear_f16act (quantize_act + GEMM + epilogue in one kernel, for small token counts)
against the oracle and against the two-call path, which it must equal bit for bit."""
import numpy as np
import pytest
import torch

from tests.gpu_util import GELU_SAME, OLAY_SAME, assert_f16, dev, f16_close, has_gpu, host

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not has_gpu(), reason="needs a GPU")]

SYM = 0


@pytest.fixture(scope="module")
def B():
    from paper_2301_12017_amd import binding
    binding.lib()
    return binding


def _case(rng, M, N, K, bias=True):
    X = rng.standard_normal((M, K)).astype(np.float32).astype(np.float16)
    W = (rng.standard_normal((N, K)) * 0.02).astype(np.float16)
    b = (rng.standard_normal(N) * 0.01).astype(np.float16) if bias else None
    return X, W, b


@pytest.mark.parametrize("M,N,K", [(128, 768, 768), (128, 2304, 768), (128, 3072, 768), (128, 768, 3072),
                                   (1, 8, 64), (33, 40, 128), (150, 264, 192), (31, 32, 4096), (257, 96, 320), (40, 2200, 832),
                                   (64, 1024, 1536), (96, 4096, 1024)])
@pytest.mark.parametrize("act", [0, 1])
def test_fused_equals_two_calls_and_oracle(B, orc, M, N, K, act):
    rng = np.random.default_rng(M * 7 + N + K + act)
    X, W, b = _case(rng, M, N, K)
    X[0, :] = 0                                                     # a constant row: scale 1, codes 0
    if M > 2:
        X[2, 5] = 60000.0                                           # one huge element: the rest of the row rounds to 0
    Q = B.quantize_weight(dev(W), SYM)
    got = host(B.linear_f16act(dev(X), Q, dev(b), act))
    A = B.quantize_act(dev(X), SYM)
    two = host(B.linear(A, Q, dev(b), act))
    assert np.array_equal(got.view(np.uint16), two.view(np.uint16))
    oa, ow = orc.quantize_act(X, SYM), orc.quantize_weight(W, SYM)
    want = orc.linear(oa, ow, SYM, 0, b, act)["out"]
    ok, ratio = f16_close(got, want)
    assert ok, ratio
    assert_f16(got, want, 1.0 if act == 0 else GELU_SAME if got.size > 200 else 0.7, f"act {act}")


def test_fused_strided_input_no_bias(B, orc):
    """X is a column slice of a wider matrix (row stride > K) and there is no bias."""
    rng = np.random.default_rng(77)
    M, N, K = 70, 136, 256
    wide = rng.standard_normal((M, 3 * K)).astype(np.float32).astype(np.float16)
    W = (rng.standard_normal((N, K)) * 0.02).astype(np.float16)
    Xd = dev(wide)[:, K:2 * K]
    assert Xd.stride(0) == 3 * K
    Q = B.quantize_weight(dev(W), SYM)
    got = host(B.linear_f16act(Xd, Q, None, 0))
    X = np.ascontiguousarray(wide[:, K:2 * K])
    want = orc.linear(orc.quantize_act(X, SYM), orc.quantize_weight(W, SYM), SYM, 0, None, 0)["out"]
    assert np.array_equal(got.view(np.uint16), want.view(np.uint16))


def test_fused_does_not_write_past_the_output(B):
    rng = np.random.default_rng(78)
    M, N, K = 37, 72, 128
    X, W, b = _case(rng, M, N, K)
    Q = B.quantize_weight(dev(W), SYM)
    buf = torch.full((M + 40, N), -7.0, dtype=torch.float16, device="cuda")
    B.linear_f16act(dev(X), Q, dev(b), 0, out=buf[:M])
    assert bool((buf[M:] == -7.0).all())
    assert bool((buf[:M] != -7.0).any())


def test_fused_non_finite_inputs_do_not_fault(B):
    rng = np.random.default_rng(79)
    X, W, b = _case(rng, 64, 64, 128)
    X[3, 7] = np.inf
    X[5, 9] = np.nan
    Q = B.quantize_weight(dev(W), SYM)
    got = host(B.linear_f16act(dev(X), Q, dev(b), 1))
    rows = np.ones(64, bool)
    rows[[3, 5]] = False
    assert np.isfinite(got[rows]).all()                             # the other tokens are unaffected


# rows of every K that is a constant of the kernel, on its tiles of 8 (long rows, up to 256 of them), 16, 32 and 32 x 64, with remainders in
# tokens and channels; and K = 640 / 2560, which are not
@pytest.mark.parametrize("M,N", [(1, 8), (9, 40), (17, 1032), (200, 264), (137, 2056)])
@pytest.mark.parametrize("K", [512, 640, 768, 1024, 1536, 2048, 2560, 3072, 4096])
def test_every_tile_of_constant_rows(B, M, N, K):
    """fp16 and packed activations, both mappings, and the INT8 sibling: exact integer sums, and the bits of the general kernel (on its
    64 x 128 tiles: the 64 x 64 ones belong to a kernel of their own for most of these K)."""
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    X = torch.randn((M, K), device="cuda", generator=g).half()
    X[:, ::7] *= 8
    W = (torch.randn((N, K), device="cuda", generator=g) * 0.02).half()
    bias = (torch.randn(N, device="cuda", generator=g) * 0.01).half()
    general, small = B.schedule_number("generic_64x128"), B.schedule_number("small_splitk")
    for mode in (0, 1):
        A, Q = B.quantize_act(X, mode), B.quantize_weight(W, mode)
        assert torch.equal(B.gemm_i32(A, Q, schedule=small), B.gemm_i32(A, Q, schedule=general))
        want = B.linear(A, Q, bias, 1, schedule=general)
        got = torch.full((M + 2, N), 7.0, dtype=torch.float16, device="cuda")
        B.linear(A, Q, bias, 1, schedule=small, out=(got[:M], None, None, None))
        assert torch.equal(got[:M].view(torch.int16), want.view(torch.int16)) and (got[M:] == 7.0).all()
        if mode == 0:
            fused = torch.full((M + 2, N), 7.0, dtype=torch.float16, device="cuda")
            B.linear_f16act(X, Q, bias, 1, out=fused[:M])
            assert torch.equal(fused.view(torch.int16), got.view(torch.int16))
    (q, s), (w8, s8) = B.quantize_rows8(X), B.quantize_rows8(W)
    P = B.gemm8_i32(q, s, w8, s8)                                   # up to 512 tiles of 32 x 32: this kernel
    assert torch.equal(P.cpu(), (q.cpu().double() @ w8.cpu().double().T).int())


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("M,N,K,group,act,with_bias", [
    (1, 8, 256, 128, 0, True), (17, 40, 1024, 128, 1, True), (33, 264, 768, 128, 0, False), (32, 32, 1024, 512, 0, True),
    (16, 96, 1152, 128, 0, True), (31, 520, 3072, 128, 1, False), (5, 72, 4096, 128, 0, True), (100, 200, 4096, 2048, 0, True),
    (301, 768, 2304, 384, 0, True)])
def test_several_weight_groups_of_a_few_tokens(mode, M, N, K, group, act, with_bias):
    """The kernel whose waves own whole weight groups (schedule 0 and 64 x 64 tiles of few tokens), in both of its tiles, with
    fewer groups than waves, as many and more: bit for bit what the 64 x 128 tiles of the general kernel give."""
    from paper_2301_12017_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    X = torch.randn((M, K), device="cuda", generator=g).half()
    X[:, ::7] *= 8
    W = (torch.randn((N, K), device="cuda", generator=g) * 0.02).half()
    bias = (torch.randn(N, device="cuda", generator=g) * 0.01).half() if with_bias else None
    A, Q = B.quantize_act(X, mode, group), B.quantize_weight(W, mode, group)
    want = B.linear(A, Q, bias, act, schedule=B.schedule_number("generic_64x128"))
    assert B.pick_schedule(A, Q) == "generic_64x64"
    got = torch.full((M + 2, N), 7.0, dtype=torch.float16, device="cuda")
    B.linear(A, Q, bias, act, out=(got[:M], None, None, None))
    assert torch.equal(got[:M].view(torch.int16), want.view(torch.int16))
    assert (got[M:] == 7.0).all()                                  # nothing behind the last row


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("K", [256, 512, 768, 1024, 1280, 1536, 2304, 4096])      # all of K at once, chunks of 256 and of 512
@pytest.mark.parametrize("M,N", [(1, 1096), (65, 264), (200, 1032)])
def test_tiles_of_64_by_64(B, mode, K, M, N):
    """One weight group on 64 x 64 tiles, remainders in tokens and channels: sums, fp16 rows (GELU), a column slice of wider packed rows
    and the fp32 rows behind a requantize, bit for bit those of the general kernel's 64 x 128 tiles."""
    g = torch.Generator(device="cuda").manual_seed(M + N + K + mode)
    X = torch.randn((M, K), device="cuda", generator=g).half()
    X[:, ::7] *= 8
    W = (torch.randn((N, K), device="cuda", generator=g) * 0.02).half()
    bias = (torch.randn(N, device="cuda", generator=g) * 0.01).half()
    A, Q = B.quantize_act(X, mode), B.quantize_weight(W, mode)
    wide = torch.randint(0, 256, (M, K // 2 + 64), dtype=torch.uint8, device="cuda", generator=g)
    wide[:, 32:32 + K // 2] = A.q
    S = B.QAct(wide, A.scale, A.zero, A.gsum, M, K, K // 2 + 64, 0, mode, q_offset_bytes=32)
    tile, general = B.schedule_number("generic_64x64"), B.schedule_number("generic_64x128")
    want = B.linear(A, Q, bias, 1, schedule=general)
    for act in (A, S):
        assert torch.equal(B.gemm_i32(act, Q, schedule=tile), B.gemm_i32(A, Q, schedule=general))
        got = torch.full((M + 2, N), 7.0, dtype=torch.float16, device="cuda")
        B.linear(act, Q, bias, 1, schedule=tile, out=(got[:M], None, None, None))
        assert torch.equal(got[:M].view(torch.int16), want.view(torch.int16)) and (got[M:] == 7.0).all()
    if N % 32 == 0 or N == 1032:
        N = N // 32 * 32
        Q = B.quantize_weight(W[:N].contiguous(), mode)
        r = [B.linear(A, Q, bias[:N].contiguous(), 0, requant=True, requant_mode=1, schedule=s) for s in (tile, general)]
        assert torch.equal(r[0].q, r[1].q) and torch.equal(r[0].scale, r[1].scale) and torch.equal(r[0].zero, r[1].zero)


@pytest.mark.parametrize("M,N,K", [(1, 8, 1280), (129, 136, 1536), (300, 1032, 1280), (257, 264, 4096), (2048, 2048, 2048)])
def test_operand_layout_tile_shared_by_two_groups_of_waves(B, M, N, K):
    """128 x 128 tiles of the operand layout with a CU each and long K, where two groups of waves share the codes of a step: sums and
    fp16 rows (without and with GELU) bit for bit those of 128 x 256 tiles, at the largest sums too; nothing behind the last row."""
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    X = torch.randn((M, K), device="cuda", generator=g).half()
    W = (torch.randn((N, K), device="cuda", generator=g) * 0.02).half()
    X[M // 2] = 3.0                                                # a row and a channel of nothing but the largest code
    W[N // 2] = -0.5
    bias = (torch.randn(N, device="cuda", generator=g) * 0.01).half()
    A, Q = B.quantize_act(X, 0, layout=1), B.quantize_weight(W, 0, layout=1)
    tile, other = B.schedule_number("olay_128x128"), B.schedule_number("olay_128x256")
    assert torch.equal(B.gemm_i32(A, Q, schedule=tile), B.gemm_i32(A, Q, schedule=other))
    for b, act in ((None, 0), (bias, 1)):
        want = B.linear(A, Q, b, act, schedule=other)
        got = torch.full((M + 2, N), 7.0, dtype=torch.float16, device="cuda")
        B.linear(A, Q, b, act, schedule=tile, out=(got[:M], None, None, None))
        assert torch.equal(got[:M].view(torch.int16), want.view(torch.int16)) and (got[M:] == 7.0).all()
