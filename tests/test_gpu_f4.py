"""The very-low-bit path on the 4-bit floating-point MFMA (weights and activations of one or two bits): the HIP kernels
through the C ABI against the oracle, element by element — int32 accumulator bit-exact, binary16 output within the same
tolerance as the int8 path, and equal to the int8 path bit for bit."""
import itertools

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from helpers import check_against_oracle, check_sampled, gpu_gemm, run_named, to_dev   # noqa: E402
from paper_2408_08554_amd import synth   # noqa: E402


def say(*a):
    print(*a, flush=True)


def run_f4(abq, c):
    pw = abq.abq_f4_pack_codes(c.p, to_dev(torch, c.W), to_dev(torch, c.w_scale), to_dev(torch, c.w_zero))
    pa = abq.abq_f4_pack_codes(c.q, to_dev(torch, c.A), to_dev(torch, c.a_scale), to_dev(torch, c.a_zero))
    y = torch.full((c.M, c.N), float("nan"), dtype=torch.float16, device="cuda")
    acc = torch.full((c.M, c.N), -7, dtype=torch.int32, device="cuda")
    abq.abq_f4_gemm(c.p, c.q, c.M, c.N, c.K, pa, pw, y=y, acc=acc)
    # without the accumulator output the kernel takes its binary32 epilogue (vector stores): the same bits
    y_only = torch.full((c.M, c.N), float("nan"), dtype=torch.float16, device="cuda")
    abq.abq_f4_gemm(c.p, c.q, c.M, c.N, c.K, pa, pw, y=y_only)
    torch.cuda.synchronize()
    assert torch.equal(y.view(torch.int16), y_only.view(torch.int16)), f"{c.name}: output differs without the accumulator"
    return y.cpu().numpy(), acc.cpu().numpy()


# one tile and less, ragged in every dimension, several workgroup tiles (32 x 64) with ragged tails, odd and even numbers
# of 128-k steps, K ending inside a step
F4_SHAPES = [(1, 1, 1), (1, 16, 128), (5, 33, 200), (16, 16, 129), (17, 130, 1000), (256, 128, 1024), (300, 520, 1000),
             (513, 257, 384), (64, 1000, 2048), (700, 300, 4096 + 64), (260, 136, 256), (31, 8, 64)]


@pytest.mark.parametrize("M,N,K", F4_SHAPES)
@pytest.mark.parametrize("p,q", list(itertools.product([1, 2], [1, 2])))
def test_f4_matmul_against_oracle(abq, p, q, M, N, K):
    c = synth.make_case(p, q, M, N, K, seed=synth.case_seed(11, p, q, M % 97, N % 89), name=f"f4 W{p}A{q} {M}x{N}x{K}")
    say(c.name)
    y, acc = run_f4(abq, c)
    check_against_oracle(c, y, acc)


def test_f4_extreme_codes(abq):
    """All codes maximal (the largest sums: K * 9), all zero, and zero-points at both ends."""
    for p, q, K in [(2, 2, 8192), (1, 2, 3000), (2, 1, 4096), (2, 2, 131072)]:   # (the last: the longest K the ABI takes)
        c = synth.make_case(p, q, 40, 70, K, seed=5, name=f"f4 max W{p}A{q} K={K}")
        c.A[:] = (1 << q) - 1
        c.W[:] = (1 << p) - 1
        c.A[1] = 0
        c.W[3] = 0
        c.a_zero[:] = np.where(np.arange(40) % 2 == 0, 0, (1 << q) - 1)
        c.w_zero[:] = np.where(np.arange(70) % 2 == 0, (1 << p) - 1, 0)
        say(c.name)
        y, acc = run_f4(abq, c)
        check_against_oracle(c, y, acc)


def test_f4_equals_the_int8_path_bitwise(abq):
    for p, q, M, N, K in [(2, 2, 300, 520, 1000), (1, 2, 64, 257, 2048), (2, 1, 1, 100, 512)]:
        c = synth.make_case(p, q, M, N, K, seed=synth.case_seed(11, p, q, M % 97, 7))
        y, acc = run_f4(abq, c)
        y8, acc8 = gpu_gemm(torch, abq, c, abq.ABQ_LAYOUT_FIELDS, abq.ABQ_LAYOUT_FIELDS)
        assert np.array_equal(acc, acc8) and np.array_equal(y.view(np.uint16), y8.view(np.uint16))


def test_f4_drops_bits_above_the_width(abq):
    """Codes with bits above `bits` set are masked, as the other packers mask them."""
    c = synth.make_case(2, 1, 20, 48, 640, seed=9)
    dirty_w = (c.W | (np.arange(c.W.size, dtype=np.uint8).reshape(c.W.shape) << 2)).astype(np.uint8)
    dirty_a = (c.A | 0xFE).astype(np.uint8)
    pw = abq.abq_f4_pack_codes(2, to_dev(torch, dirty_w), to_dev(torch, c.w_scale), to_dev(torch, c.w_zero))
    pa = abq.abq_f4_pack_codes(1, to_dev(torch, dirty_a), to_dev(torch, c.a_scale), to_dev(torch, c.a_zero))
    y, acc = abq.abq_f4_gemm(2, 1, c.M, c.N, c.K, pa, pw, want_acc=True)
    torch.cuda.synchronize()
    check_against_oracle(c, y.cpu().numpy(), acc.cpu().numpy())


def test_f4_large_tile_sampled(abq):
    """Two workgroups of 128 x 128 on every compute unit, K of eight steps (two turns of the ring), the last one short; then 256 x 256 tiles with
    two bands of row tiles, the second of fewer: sampled outputs."""
    for M, N, K in [(1024, 8192, 1000), (2600, 3300, 640)]:
        c = synth.make_case(2, 2, M, N, K, seed=synth.case_seed(11, 2, 2, 55, 66), name=f"f4 W2A2 {M}x{N}x{K}")
        say(c.name)
        y, acc = run_f4(abq, c)
        check_sampled(c, y, acc)


@pytest.mark.parametrize("p,q", [(2, 2), (1, 1)])
def test_f4_config5_prefill_shape_sampled(abq, p, q):
    """M = 2048 on the LLaMA-13B up-projection, the launch the bench times: sampled outputs against the oracle."""
    c = synth.config5(p, q, 0, 3)
    say(c.name)
    y, acc = run_f4(abq, c)
    check_sampled(c, y, acc)


# Every workgroup shape by the rule, ragged rows and channels (rows of Y on and off 16-byte boundaries), K of one block of 128, of an odd and an even
# number of them, of fewer and more steps than the ring has places
@pytest.mark.parametrize("waves,M,N,K", [("2, 4, 8, 4", 1029, 7195, 59), ("2, 4, 8, 4", 904, 8400, 257), ("2, 4, 8, 4", 905, 8412, 406), ("2, 4, 8, 4", 901, 8213, 1300),
                                         ("2, 4, 4, 2", 196, 8504, 261), ("2, 4, 4, 2", 195, 8313, 401), ("2, 4, 4, 2", 197, 8333, 1700),
                                         ("2, 2, 4, 4", 513, 7183, 84), ("2, 2, 4, 4", 705, 5408, 129), ("2, 2, 4, 4", 518, 7309, 385), ("2, 2, 4, 4", 459, 8258, 517),
                                         ("1, 4, 4, 2", 97, 8274, 69), ("1, 4, 4, 2", 105, 8444, 131), ("1, 4, 4, 2", 100, 8855, 1175),
                                         ("1, 2, 2, 2", 19, 203, 103), ("1, 2, 2, 2", 18, 201, 204), ("1, 2, 2, 2", 37, 232, 347), ("1, 2, 2, 2", 24, 214, 2306)])
@pytest.mark.parametrize("p,q", [(2, 2), (1, 2)])
def test_f4_shapes_by_rule(abq, p, q, waves, M, N, K):
    c = synth.make_case(p, q, M, N, K, seed=7600 + p, name=f"f4 {waves} W{p}A{q} {M}x{N}x{K}")
    say(c.name)
    c.W[::5], c.A[::7] = (1 << p) - 1, (1 << q) - 1
    pw = abq.abq_f4_pack_codes(p, to_dev(torch, c.W), to_dev(torch, c.w_scale), to_dev(torch, c.w_zero))
    pa = abq.abq_f4_pack_codes(q, to_dev(torch, c.A), to_dev(torch, c.a_scale), to_dev(torch, c.a_zero))
    _, names = run_named(torch, lambda: abq.abq_f4_gemm(p, q, M, N, K, pa, pw))
    assert len(names) == 1 and f"f4_gemm_kernel<{waves}, " in names[0], names
    y, acc = run_f4(abq, c)
    (check_against_oracle if M * N * K < 2e8 else check_sampled)(c, y, acc)
