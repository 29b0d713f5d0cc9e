"""The K-split prefill kernel (more than 16 rows over few output tiles): every workgroup shape at the edges of its tiles and of K,
from packed and from unpacked rows, bit for bit against the tiled and streaming kernels (which a plan-table entry brings back)
and against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2408_08554_amd import synth
from helpers import check_against_oracle, check_g128, check_sampled, run_named, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

FIELDS, G128 = 2, 4
# rows, channels: 32 x 16, 32 x 32, 64 x 32 and 64 x 64 tiles on 256 compute units, whole and ragged in both directions (64 x 64: rows enough
# that codes of any length are read as they are)
SHAPES = {"32x16": [(17, 40), (33, 1003), (96, 64)], "32x32": [(50, 2100), (64, 4096)], "64x32": [(70, 4001), (257, 1600)],
          "64x64": [(129, 4100), (300, 3001), (520, 1601)]}
KERNEL = {"32x16": "KsShape<2, 1,", "32x32": "KsShape<2, 2,", "64x32": "KsShape<4, 2,", "64x64": "KsShape<4, 4,"}


def other_kernel(abq, c, call):
    """The same call while a plan-table entry asks for one of the other kernels."""
    abq.abq_plan_set(c.p, c.q, c.M, c.N, c.K, tiled_mt=4, skinny_waves=1)
    try:
        return call()
    finally:
        abq.abq_plan_set(c.p, c.q, c.M, c.N, c.K)


# K: one load, off a 16-byte boundary, one phase of 256 past and short of whole super-chunks, waves with one to five phases
@pytest.mark.parametrize("K", [16, 255, 700, 2053, 3072, 3077, 4096, 4620])
@pytest.mark.parametrize("shape", list(SHAPES))
@pytest.mark.parametrize("p,q", [(1, 8), (2, 3), (3, 8), (4, 8), (5, 4), (6, 6), (7, 8), (8, 8), (8, 7)])
def test_ksplit_equals_the_other_kernels(abq, p, q, shape, K):
    if shape == "64x64" and K < 3072:
        pytest.skip("64 x 64 tiles are taken from K = 3072")
    unpacked = 0
    for i, (M, N) in enumerate(SHAPES[shape]):
        if M <= 48 and K >= 3072:
            M += 32   # (fewer rows are the streaming kernel's)
        c = synth.make_case(p, q, M, N, K, seed=7000 + 10 * p + i, name=f"ksplit W{p}A{q} {M}x{N}x{K}")
        print(c.name, flush=True)
        a, sa, za = to_dev(torch, c.A), to_dev(torch, c.a_scale), to_dev(torch, c.a_zero)
        pw = abq.abq_pack_weights(p, to_dev(torch, c.W), to_dev(torch, c.w_scale), to_dev(torch, c.w_zero))
        pa = abq.abq_pack_act_codes(q, a, sa, za)
        calls = [lambda acc: abq.abq_gemm_act_codes(p, q, M, N, K, a, sa, za, pw, FIELDS, want_acc=acc),
                 lambda acc: abq.abq_gemm(p, q, M, N, K, pa, FIELDS, pw, FIELDS, want_acc=acc)]
        (y0, acc0), names = run_named(torch, lambda: other_kernel(abq, c, lambda: calls[1](True)))
        assert len(names) == 1 and ("tiled_kernel" in names[0] or "skinny_kernel" in names[0]), names
        for call in calls:
            (y, acc), names = run_named(torch, lambda: call(True))
            y2, _ = call(False)
            assert f"ksplit_kernel<{p}, abq::{KERNEL[shape]}" in names[-1] and (len(names) == 1 or call is calls[0]), names
            unpacked += call is calls[0] and len(names) == 1
            assert torch.equal(acc, acc0) and torch.equal(y.view(torch.int16), y0.view(torch.int16)) and torch.equal(y2.view(torch.int16), y0.view(torch.int16))
        check = check_against_oracle if M * N * K < 2e8 else check_sampled
        check(c, y0.cpu().numpy(), acc0.cpu().numpy())
    assert unpacked >= (1 if shape == "64x64" else len(SHAPES[shape]))


@pytest.mark.parametrize("p,q", [(1, 8), (3, 4), (4, 8), (5, 8), (6, 8), (7, 8), (8, 5)])
@pytest.mark.parametrize("shape,K", [(s, K) for s in SHAPES for K in (16, 130, 1000, 2064, 4096, 6160) if s != "64x64" or K >= 2048])
def test_ksplit_per_group_weights(abq, p, q, shape, K):
    if shape == "64x64" and p <= 6:
        pytest.skip("64 x 64 tiles of per-group weights are taken for p = 7, 8")
    M, N = SHAPES[shape][1]
    c = synth.make_case(p, q, M, N, K, seed=7100 + p, name=f"ksplit g128 W{p}A{q} {M}x{N}x{K}")
    print(c.name, flush=True)
    sh, zg = synth.group_quant_params(c)
    if M * N * K > 1e9 and p not in (4, 7, 8):
        pytest.skip("the large sizes run for three widths")
    top = (1 << p) - 1
    zg[:, 0::2], c.W[0::3], c.A[0::4], c.a_zero[1::3] = top, 0, (1 << q) - 1, 0   # ends of the ranges against each other
    c.a_scale[:] = np.float32(2e-4 * 1000 / max(K, 1000))
    a, sa, za = to_dev(torch, c.A), to_dev(torch, c.a_scale), to_dev(torch, c.a_zero)
    pw = abq.abq_pack_weights_g128(p, to_dev(torch, c.W), to_dev(torch, sh.view(np.float16)), to_dev(torch, zg))
    pa = abq.abq_pack_act_codes(q, a, sa, za)
    calls = [lambda: abq.abq_gemm(p, q, M, N, K, pa, FIELDS, pw, G128)[:1], lambda: abq.abq_gemm_act_codes(p, q, M, N, K, a, sa, za, pw, G128)[:1]]
    ys = []
    for call in calls:
        out, names = run_named(torch, call)
        assert f"ksplit_kernel<{p}, abq::{KERNEL[shape]}" in names[-1] and len(names) == 1 + (call is calls[1] and K % 16 != 0), names
        ys.append(out[0].cpu().numpy())
    assert np.array_equal(ys[0].view(np.uint16), ys[1].view(np.uint16))   # packed and unpacked rows: one order of sums
    # the tiled kernel: the same rows over and over, until no compute unit would get one tile only
    M2 = max(M, 64 * (256 // ((N + 63) // 64) + 1))
    rows = torch.arange(M2, device="cuda") % M
    pa2 = abq.abq_pack_act_codes(q, a[rows].contiguous(), sa[rows].contiguous(), za[rows].contiguous())
    out, names = run_named(torch, lambda: abq.abq_gemm(p, q, M2, N, K, pa2, FIELDS, pw, G128)[:1])
    assert len(names) == 1 and "tiled_g128_kernel" in names[0], names
    ys.append(out[0][:M].cpu().numpy())
    for y in ys[1:] if M * N * K < 5e8 else ys[1:2]:
        check_g128(c, sh, zg, y)
    ref = ys[0].astype(np.float64)   # the same integers summed in another order: an output may round to the neighbouring binary16, at most 2^-10 of it
    assert np.linalg.norm(ys[2] - ref) <= 2.0 ** -10 * np.linalg.norm(ref)


@pytest.mark.parametrize("p,q,M,N,K", [(4, 8, 40, 130, 1000), (8, 6, 100, 2051, 528)])
def test_ksplit_codes_past_q_bits_and_requant(abq, p, q, M, N, K):
    """Codes with bits above q set are masked as the packers mask them; the requantizing epilogue and the static call."""
    c = synth.make_case(p, q, M, N, K, seed=7200, name=f"ksplit W{p}A{q} {M}x{N}x{K}")
    print(c.name, flush=True)
    a, sa, za = to_dev(torch, c.A | (0xFF & ~((1 << q) - 1))), to_dev(torch, c.a_scale), to_dev(torch, c.a_zero)
    pw = abq.abq_pack_weights(p, to_dev(torch, c.W), to_dev(torch, c.w_scale), to_dev(torch, c.w_zero))
    so, zo = torch.rand(M, device="cuda") + 0.5, torch.randint(0, 256, (M,), dtype=torch.int32, device="cuda")
    static = torch.empty((M, N), dtype=torch.float16, device="cuda")
    abq.abq_gemm_act_codes_static(p, q, M, N, K, a, sa, za, pw, FIELDS, static)
    run = lambda: abq.abq_gemm_act_codes_requant(p, q, M, N, K, a, sa, za, pw, FIELDS, 8, so, zo)
    codes, y = run()[:2]
    codes0, y0 = other_kernel(abq, c, run)[:2]
    assert torch.equal(codes, codes0) and torch.equal(y.view(torch.int16), y0.view(torch.int16)) and torch.equal(static.view(torch.int16), y0.view(torch.int16))
    check_against_oracle(c, y.cpu().numpy(), None)


@pytest.mark.parametrize("raw", [False, True], ids=["packed", "codes"])
@pytest.mark.parametrize("N,kernel", [(8128, "skinny_kernel"), (8129, "ksplit_kernel"), (8192, "ksplit_kernel")])
def test_streaming_kernel_is_left_the_rows_that_it_takes(abq, N, kernel, raw):
    """32 x 32 tiles of wide weights and long K are left to the streaming kernel; where it does not run (above 8128 channels) the prefill
    kernel would take them at up to twice the time."""
    p, q, M, K = 6, 8, 32, 3072
    c = synth.make_case(p, q, M, N, K, seed=7300, name=f"ksplit or streaming W{p}A{q} {M}x{N}x{K}")
    print(c.name, raw, flush=True)
    a, sa, za = to_dev(torch, c.A), to_dev(torch, c.a_scale), to_dev(torch, c.a_zero)
    pw = abq.abq_pack_weights(p, to_dev(torch, c.W), to_dev(torch, c.w_scale), to_dev(torch, c.w_zero))
    pa = abq.abq_pack_act_codes(q, a, sa, za)
    out, names = run_named(torch, lambda: abq.abq_gemm_act_codes(p, q, M, N, K, a, sa, za, pw, FIELDS, want_acc=True) if raw
                           else abq.abq_gemm(p, q, M, N, K, pa, FIELDS, pw, FIELDS, want_acc=True))
    assert len(names) == 1 and kernel in names[0], names
    check_sampled(c, out[0].cpu().numpy(), out[1].cpu().numpy())


KS44 = "ksplit_kernel<%d, abq::KsShape<4, 4"


@pytest.mark.parametrize("p,M,N,K,kernels", [(4, 57, 11008, 5120, ["act_code", KS44 % 4]), (2, 38, 12880, 3296, ["act_code", KS44 % 2]),
                                             (8, 38, 12880, 3296, ["act_code", "tiled_kernel"]), (8, 57, 11008, 4620, ["act_code", KS44 % 8]),
                                             (8, 199, 2672, 3072, [KS44 % 8]), (3, 199, 4000, 3076, ["act_code", KS44 % 3]),
                                             (3, 400, 2000, 3076, [KS44 % 3]), (3, 400, 2000, 3075, ["act_code", KS44 % 3]), (3, 520, 1600, 3075, [KS44 % 3])])
def test_codes_on_64x64_tiles(abq, p, M, N, K, kernels):
    """Where codes go as they are and where they are packed first, and that the result is the same bits."""
    q = 8 if p < 8 else 7
    c = synth.make_case(p, q, M, N, K, seed=7400 + p, name=f"codes on 64 x 64 W{p}A{q} {M}x{N}x{K}")
    print(c.name, flush=True)
    a, sa, za = to_dev(torch, c.A), to_dev(torch, c.a_scale), to_dev(torch, c.a_zero)
    pw = abq.abq_pack_weights(p, to_dev(torch, c.W), to_dev(torch, c.w_scale), to_dev(torch, c.w_zero))
    pa = abq.abq_pack_act_codes(q, a, sa, za)
    out, names = run_named(torch, lambda: abq.abq_gemm_act_codes(p, q, M, N, K, a, sa, za, pw, FIELDS, want_acc=True))
    assert len(names) == len(kernels) and all(k in n for k, n in zip(kernels, names)), names
    y0, acc0 = other_kernel(abq, c, lambda: abq.abq_gemm(p, q, M, N, K, pa, FIELDS, pw, FIELDS, want_acc=True))
    assert torch.equal(out[1], acc0) and torch.equal(out[0].view(torch.int16), y0.view(torch.int16))
    check_sampled(c, y0.cpu().numpy(), acc0.cpu().numpy())


# 40 rows: the streaming kernel is the other choice (K of four super-chunks: eight waves do not fit); 128 rows: the prefill kernel
@pytest.mark.parametrize("g128", [False, True], ids=["per_channel", "per_group"])
@pytest.mark.parametrize("M,plan,kernel", [(40, dict(skinny_waves=4), "skinny_kernel"), (40, dict(skinny_waves=8), "ksplit_kernel"),
                                           (40, dict(skinny_kgroups=1), "skinny_kernel"), (40, dict(tiled_mt=4, tiled_ntw=1), "ksplit_kernel"),
                                           (128, dict(skinny_waves=4), "ksplit_kernel"), (128, dict(tiled_band=2), "ksplit_kernel"),
                                           (128, dict(tiled_wd=4), "ksplit_kernel"), (128, dict(tiled_mt=8), "tiled_kernel"),
                                           (128, dict(tiled_ntw=2), "tiled_kernel"), (128, dict(direct_r=1), "ksplit_kernel")])
def test_plan_entries_that_do_not_apply_leave_the_rules_kernel(abq, M, plan, kernel, g128):
    """A table entry takes a problem off the K-split kernel only where it asks for a shape of the kernel that runs instead: not by a knob of
    a kernel that does not take the problem, by a value that does not fit, by a refinement alone, or on per-group blobs."""
    p, q, N, K = 4, 8, 600, 2048
    c = synth.make_case(p, q, M, N, K, seed=7500 + M, name=f"ksplit under {plan} W{p}A{q} {M}x{N}x{K}")
    print(c.name, g128, flush=True)
    a, sa, za = to_dev(torch, c.A), to_dev(torch, c.a_scale), to_dev(torch, c.a_zero)
    if g128:
        sh, zg = synth.group_quant_params(c)
        pw, layout, kernel = abq.abq_pack_weights_g128(p, to_dev(torch, c.W), to_dev(torch, sh.view(np.float16)), to_dev(torch, zg)), G128, "ksplit_kernel"
    else:
        pw, layout = abq.abq_pack_weights(p, to_dev(torch, c.W), to_dev(torch, c.w_scale), to_dev(torch, c.w_zero)), FIELDS
    pa = abq.abq_pack_act_codes(q, a, sa, za)
    calls = [lambda: abq.abq_gemm(p, q, M, N, K, pa, FIELDS, pw, layout)[0], lambda: abq.abq_gemm_act_codes(p, q, M, N, K, a, sa, za, pw, layout)[0]]
    y0 = [call() for call in calls]
    try:
        abq.abq_plan_set(p, q, M, N, K, **plan)
        for call, y in zip(calls, y0):
            out, names = run_named(torch, call)
            assert kernel in names[-1] and len(names) == 1 + (kernel == "tiled_kernel" and call is calls[1]), (plan, names)
            assert torch.equal(out.view(torch.int16), y.view(torch.int16))
    finally:
        abq.abq_plan_set(p, q, M, N, K)
