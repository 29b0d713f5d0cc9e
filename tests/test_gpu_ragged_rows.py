"""Rows of activations of any length on the device: the row kernels' workgroup choices and tails, and the decode kernel
that reads unpacked rows starting at any byte, against the oracle (codes, sums, padding and accumulators bit for bit)."""
import numpy as np
import pytest

import oracle
from paper_2408_08554_amd import synth
from helpers import check_against_oracle, check_g128, check_sampled, gpu_gemm, gpu_gemm_fused, run_named, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

FIELDS = 2
# one K per workgroup choice, off and on a vector, one element past and short of it
LENGTHS = [1, 7, 9, 17, 504, 513, 1023, 2049, 4091, 4104, 8199, 12289, 16385, 32761, 33000]


@pytest.mark.parametrize("K", LENGTHS)
@pytest.mark.parametrize("M,q", [(3, 8), (300, 5)])
def test_row_packers_any_length(abq, M, q, K):
    if M > 3 and K > 13000:
        M = 260
    print("rows", M, q, K, flush=True)
    x = synth.act_fp16(5000 + K, M, K)
    x[1] = 0
    c = synth.make_case(2, q, M, 16, K, seed=5100 + K)
    ref_codes, ref_scale, ref_zero = oracle.quant_act(x, q)
    Kp, oa = (K + 511) // 512 * 512, 128 if q == 8 else 0
    off = 256 + (M * 16 + 255) // 256 * 256
    for packed, codes, scale, zero in ((abq.abq_quant_pack_act(q, to_dev(torch, x)), ref_codes, ref_scale, ref_zero),
                                       (abq.abq_pack_act_codes(q, to_dev(torch, c.A), to_dev(torch, c.a_scale), to_dev(torch, c.a_zero)),
                                        c.A, c.a_scale, c.a_zero)):
        _, sc, zp, sm = abq.abq_unpack_act(q, M, K, FIELDS, packed, FIELDS)
        rows = packed.cpu().numpy()[off:off + M * Kp].view(np.int8).reshape(M, Kp)
        assert np.array_equal(rows[:, :K].astype(np.int64) + oa, codes.astype(np.int64))
        assert not rows[:, K:].any()                                          # padding is zero bytes
        assert np.array_equal(sc.cpu().numpy(), scale) and np.array_equal(zp.cpu().numpy(), zero)
        assert np.array_equal(sm.cpu().numpy().astype(np.int64), codes.astype(np.int64).sum(axis=1))


@pytest.mark.parametrize("M", [1, 2, 5, 16])
@pytest.mark.parametrize("p,q,N,K", [(4, 8, 40, 17), (3, 5, 33, 31), (8, 8, 20, 1000), (1, 3, 50, 4091), (7, 7, 16, 2062), (2, 8, 31, 13001)])
def test_fused_decode_of_rows_of_any_length(abq, M, p, q, N, K):
    c = synth.make_case(p, q, M, N, K, seed=5200 + M + K, name=f"W{p}A{q} {M}x{N}x{K}")
    print(c.name, flush=True)
    y, acc = gpu_gemm_fused(torch, abq, c, FIELDS)
    check_against_oracle(c, y, acc)


@pytest.mark.parametrize("p,M", [(4, 2), (8, 3), (3, 12)])
def test_grouped_short_and_ragged_rows_equal_single_calls(abq, p, M):
    q, cases, problems = 8, [], []
    for i, (N, K) in enumerate([(64, 1120), (40, 1120), (30, 3001), (64, 700)]):
        c = synth.make_case(p, q, M, N, K, seed=5300 + i, name=f"grouped W{p}A{q} {M}x{N}x{K}")
        cases.append(c)
        problems.append({"N": N, "K": K, "packed_w": abq.abq_pack_weights(p, to_dev(torch, c.W), to_dev(torch, c.w_scale), to_dev(torch, c.w_zero)),
                         "a_codes": to_dev(torch, c.A), "a_scale": to_dev(torch, c.a_scale), "a_zero": to_dev(torch, c.a_zero),
                         "y": torch.empty((M, N), dtype=torch.float16, device="cuda")})
    print("grouped", p, M, flush=True)
    arr = abq.make_problems(problems)
    need = abq.abq_gemm_grouped_workspace_bytes(p, q, M, arr, FIELDS, FIELDS)
    abq.abq_gemm_grouped(p, q, M, arr, FIELDS, FIELDS, workspace=torch.empty(need, dtype=torch.uint8, device="cuda") if need else None)
    torch.cuda.synchronize()
    for c, d in zip(cases, problems):
        y1, _ = gpu_gemm_fused(torch, abq, c, FIELDS)
        assert np.array_equal(d["y"].cpu().numpy().view(np.uint16), y1.view(np.uint16)), c.name


@pytest.mark.parametrize("p,K", [(4, 1000), (3, 4091), (2, 9001)])
def test_g128_one_row_of_any_length(abq, p, K):
    N, q = 40, 8
    c = synth.make_case(p, q, 1, N, K, seed=5400 + K, name=f"g128 W{p}A{q} 1x{N}x{K}")
    sh, zg = synth.group_quant_params(c)
    pw = abq.abq_pack_weights_g128(p, to_dev(torch, c.W), to_dev(torch, sh.view(np.float16)), to_dev(torch, zg))
    print(c.name, flush=True)
    y, _ = abq.abq_gemm_act_codes(p, q, 1, N, K, to_dev(torch, c.A), to_dev(torch, c.a_scale), to_dev(torch, c.a_zero), pw, abq.ABQ_LAYOUT_FIELDS_G128)
    torch.cuda.synchronize()
    check_g128(c, sh, zg, y.cpu().numpy())


def _graph_us(fn, count=8):
    """Device time of one call, from replays of a graph of `count` calls (the fastest of five)."""
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        fn()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        for _ in range(count):
            fn()
    best = float("inf")
    for _ in range(6):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record(), g.replay(), b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / count)
    return best


@pytest.mark.parametrize("K", [32768 + 16, 53248, 65536 + 9, 131072 - 5, 131072])
def test_quantizer_of_the_longest_rows(abq, K):
    """Rows of more than 32768 halves: codes, sums and padding, and the time of such a row against that of the longest row below."""
    M, q = 3, 8
    print("long rows", K, flush=True)
    x = synth.act_fp16(5500 + K, M, K)
    codes, scale, zero = oracle.quant_act(x, q)
    xd = to_dev(torch, x)
    packed = abq.abq_quant_pack_act(q, xd)
    _, sc, zp, sm = abq.abq_unpack_act(q, M, K, FIELDS, packed, FIELDS)
    Kp, off = (K + 511) // 512 * 512, 256 + (M * 16 + 255) // 256 * 256
    rows = packed.cpu().numpy()[off:off + M * Kp].view(np.int8).reshape(M, Kp)
    assert np.array_equal(rows[:, :K].astype(np.int64) + 128, codes.astype(np.int64)) and not rows[:, K:].any()
    assert np.array_equal(sc.cpu().numpy(), scale) and np.array_equal(zp.cpu().numpy(), zero)
    assert np.array_equal(sm.cpu().numpy().astype(np.int64), codes.astype(np.int64).sum(axis=1))
    # one workgroup per row either way, so the time goes with the row at most (a fixed part keeps it below); element by element, a
    # row just above 32768 took ten times the one just below
    ref = torch.from_numpy(x[:, :32768].copy()).cuda()
    out = torch.empty_like(packed)
    longest, below = _graph_us(lambda: abq.abq_quant_pack_act(q, xd, out=out)), _graph_us(lambda: abq.abq_quant_pack_act(q, ref, out=out))
    assert longest < 2.0 * below * K / 32768, f"{longest:.1f} us against {below:.1f} us for 32768"


@pytest.mark.parametrize("p,M,N,K,one_kernel", [
    (2, 1, 13824, 5118, True), (5, 1, 13824, 5118, True),                                # one row
    (1, 4, 13824, 5124, True), (1, 8, 13824, 5124, False),                               # up to four rows on dword boundaries
    (4, 16, 4096, 9212, True), (4, 16, 4096, 9220, False),                               # else 144 KiB of A per compute unit
    (4, 12, 4096, 4090, True), (4, 13, 4096, 4090, False), (8, 16, 1024, 3070, True), (8, 16, 1024, 3074, False),   # 48 KiB
    (2, 2, 13824, 5118, True), (2, 3, 13824, 5118, False), (2, 16, 13824, 5118, False)])
def test_kernel_of_ragged_rows(abq, p, M, N, K, one_kernel):
    """Rows that are no whole number of 16-byte vectors go to the direct kernel as they are only while it reads few bytes of them;
    the others are packed first and run on the kernel of packed rows.  Both give the oracle's result."""
    c = synth.make_case(p, 8, M, N, K, seed=5600 + M + K, name=f"W{p}A8 {M}x{N}x{K}")
    print(c.name, flush=True)
    lib = abq.load()
    y1, _ = gpu_gemm(torch, abq, c, FIELDS, FIELDS, want_acc=False)
    packed_kernel = lib.abq_last_decode_kernel()
    y, acc = gpu_gemm_fused(torch, abq, c, FIELDS)
    assert lib.abq_last_decode_kernel() == (1 if one_kernel else packed_kernel)
    check_sampled(c, y, acc)
    assert np.array_equal(y.view(np.uint16), y1.view(np.uint16))


def _kernels(fn):
    return run_named(torch, fn)[1]


@pytest.mark.parametrize("K", [4090, 4096])
def test_plan_entry_holds_for_unpacked_rows_of_any_length(abq, K):
    """A table entry's super-chunks per wave (the kernel's third parameter) and its choice of another kernel, off and on a vector."""
    p, q, M, N = 4, 8, 1, 64
    c = synth.make_case(p, q, M, N, K, seed=5700 + K)
    print("plan", K, flush=True)
    pw = abq.abq_pack_weights(p, to_dev(torch, c.W), to_dev(torch, c.w_scale), to_dev(torch, c.w_zero))
    a = (to_dev(torch, c.A), to_dev(torch, c.a_scale), to_dev(torch, c.a_zero))
    try:
        for r in (1, 2, 4, -1):
            abq.abq_plan_set(p, q, M, N, K, direct_r=r)
            names = _kernels(lambda: abq.abq_gemm_act_codes(p, q, M, N, K, *a, pw, FIELDS))
            if r > 0:
                assert len(names) == 1 and f"direct_kernel<{p}, 1, {r}, true" in names[0], (r, names)
            else:
                assert "skinny_kernel" in names[-1], (r, names)
    finally:
        abq.abq_plan_clear()


@pytest.mark.parametrize("p,M,K,count,packed,direct", [
    (2, 16, 5118, 4, False, True), (2, 16, 5118, 6, False, False),        # off dword boundaries: 400 KiB of A per compute unit
    (2, 16, 5124, 15, False, True), (2, 16, 5124, 17, False, False),      # on them: 1280 KiB
    (1, 16, 5124, 12, False, True), (1, 16, 5124, 14, False, False),      # W1: 1024 KiB
    (8, 3, 1120, 4, False, True), (8, 3, 1120, 4, True, True)])           # short rows of the widest weights
def test_route_of_groups_the_streaming_launch_does_not_fit(abq, p, M, K, count, packed, direct):
    """Direct launches while the group reads few bytes of A and no member has a plan entry, else one call after the other; the same
    results either way.  (4096 channels: one tile per compute unit.)"""
    q, N = 8, 4096
    c = synth.make_case(p, q, M, N, K, seed=5800 + K + M, name=f"grouped W{p}A{q} {count} x {M}x{N}x{K}")
    print(c.name, packed, flush=True)
    pw = abq.abq_pack_weights(p, to_dev(torch, c.W), to_dev(torch, c.w_scale), to_dev(torch, c.w_zero))
    a = (to_dev(torch, c.A), to_dev(torch, c.a_scale), to_dev(torch, c.a_zero))
    acts = {"packed_act": abq.abq_pack_act_codes(q, *a)} if packed else dict(zip(("a_codes", "a_scale", "a_zero"), a))
    problems = [{"N": N, "K": K, "packed_w": pw, **acts, "y": torch.zeros((M, N), dtype=torch.float16, device="cuda")} for _ in range(count)]
    arr = abq.make_problems(problems)
    need = abq.abq_gemm_grouped_workspace_bytes(p, q, M, arr, FIELDS, FIELDS)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda") if need else None
    run = lambda: abq.abq_gemm_grouped(p, q, M, arr, FIELDS, FIELDS, workspace=ws)
    grouped = lambda names: all("direct_kernel" in n and ", true, false>" in n for n in names) and len(names) == (count + 7) // 8   # (GROUPED)
    names = _kernels(run)
    assert grouped(names) == direct, names
    y1, _ = gpu_gemm_fused(torch, abq, c, FIELDS, want_acc=False)
    for d in problems:
        assert np.array_equal(d["y"].cpu().numpy().view(np.uint16), y1.view(np.uint16))
        d["y"].zero_()
    if direct:
        try:
            abq.abq_plan_set(p, q, M, N, K, direct_r=-1)
            names = _kernels(run)
        finally:
            abq.abq_plan_clear()
        assert not grouped(names) and sum("skinny_kernel" in n for n in names) == count, names
        for d in problems:
            assert np.array_equal(d["y"].cpu().numpy().view(np.uint16), y1.view(np.uint16))


@pytest.mark.parametrize("M", [4, 260])
@pytest.mark.parametrize("K", [7, 513, 4096, 4091, 12289, 16392, 33000, 53248])
def test_halves_that_are_no_numbers(abq, M, K):
    """A NaN moves no row's range and gets the code of zero, an infinity makes the step infinite and every code zero: the same from
    the row kernels, the kernel of blobs with planes and the producers."""
    q, rng = 8, np.random.default_rng(5900 + K)
    if M > 4 and K > 13000:
        pytest.skip("the long rows' kernels do not depend on M")
    print("NaN", M, K, flush=True)
    x = synth.act_fp16(5900 + K, M, K)
    x[0, rng.random(K) < 0.3] = np.nan
    x[1], x[2, K - 1], x[3, 0] = np.nan, np.nan, -np.nan
    codes, scale, zero = oracle.quant_act(np.where(np.isnan(x), np.float16(0), x), q)
    for layout in (FIELDS, 3):
        got = [t.cpu().numpy() for t in abq.abq_unpack_act(q, M, K, layout, abq.abq_quant_pack_act(q, to_dev(torch, x), layout), FIELDS)]
        assert np.array_equal(got[0], codes) and np.array_equal(got[1], scale) and np.array_equal(got[2], zero), layout
        assert np.array_equal(got[3].astype(np.int64), codes.astype(np.int64).sum(axis=1))
    up = synth.act_fp16(5901 + K, M, K)
    c, sc, zp, h = (t.cpu().numpy() for t in abq.abq_silu_mul_quant_act(q, to_dev(torch, x), to_dev(torch, up), want_h=True))
    assert np.array_equal(np.isnan(h), np.isnan(x))
    codes, scale, zero = oracle.quant_act(np.where(np.isnan(h), np.float16(0), h), q)
    assert np.array_equal(c, codes) and np.array_equal(sc, scale) and np.array_equal(zp, zero)
    x = synth.act_fp16(5902 + K, M, K)
    x[0, 3], x[1, K - 1], x[2, 1], x[2, 2] = np.inf, -np.inf, np.inf, -np.inf
    a, b = ([t.cpu().numpy() for t in abq.abq_unpack_act(q, M, K, layout, abq.abq_quant_pack_act(q, to_dev(torch, x), layout), FIELDS)] for layout in (FIELDS, 3))
    assert all(np.array_equal(s, t) for s, t in zip(a, b)) and np.isinf(a[1][:3]).all() and not a[0][:3].any()


@pytest.mark.parametrize("M", [3, 260])
@pytest.mark.parametrize("K", [1023, 2049, 4091, 4104, 6149, 8199, 12289, 16384, 32761, 32768, 32776])
def test_producers_of_any_length(abq, M, K):
    """RMSNorm with and without the residual (its sum over the residual itself) and SiLU * up over the row kernels' workgroup choices, few
    rows and many, on a vector and off it, and one row past the longest of them."""
    q, rng = 8, np.random.default_rng(6000 + K)
    distinct = min(M, 5)                              # (the oracle takes its time: the other rows repeat these)
    rows = np.arange(M) % distinct
    x, res, up = (synth.act_fp16(6000 + 3 * K + i, distinct, K) for i in range(3))
    gamma = (1.0 + 0.2 * rng.standard_normal(K)).astype(np.float16)
    x[1], res[1] = 0, 0
    print("producers", M, K, flush=True)
    dev = lambda a: to_dev(torch, a[rows])
    bits = lambda t: t.cpu().numpy().view(np.uint16)

    def check(got, produced):
        codes, scale, zero, out = got
        c, s, z = oracle.quant_act(produced, q)
        assert np.array_equal(bits(out), produced.view(np.uint16)[rows]) and np.array_equal(codes.cpu().numpy(), c[rows])
        assert np.array_equal(scale.cpu().numpy(), s[rows]) and np.array_equal(zero.cpu().numpy(), z[rows])

    g = to_dev(torch, gamma)
    check(abq.abq_rmsnorm_quant_act(q, dev(x), g, 1e-5, want_y=True), oracle.rmsnorm_half(x, gamma, 1e-5))
    h = oracle.add_half(x, res)
    r = dev(res)
    *got, h_out, y = abq.abq_add_rmsnorm_quant_act(q, dev(x), r, g, 1e-5, want_y=True, sum_out=r)
    assert h_out.data_ptr() == r.data_ptr() and np.array_equal(bits(r), h.view(np.uint16)[rows])
    check((*got, y), oracle.rmsnorm_half(h, gamma, 1e-5))
    check(abq.abq_silu_mul_quant_act(q, dev(x), dev(up), want_h=True), oracle.silu_mul_half(x, up))


@pytest.mark.parametrize("M", [5, 8, 9, 16])
@pytest.mark.parametrize("p,q,N,K", [(4, 8, 70, 10320), (8, 7, 90, 5872), (2, 8, 4100, 4096), (6, 8, 33, 9808), (3, 5, 40, 7001), (5, 8, 300, 6144), (7, 8, 4111, 3100)])
def test_decode_rows_in_lane_order(abq, p, q, M, N, K):
    """Eight and sixteen operand rows on enough K and tiles that the direct kernel loads the rows of A in lane order."""
    c = synth.make_case(p, q, M, N, K, seed=5900 + M + p, name=f"W{p}A{q} {M}x{N}x{K}")
    print(c.name, flush=True)
    for y, acc in (gpu_gemm_fused(torch, abq, c, FIELDS), gpu_gemm(torch, abq, c, FIELDS, FIELDS)):
        (check_against_oracle if M * N * K < 2e8 else check_sampled)(c, y, acc)


@pytest.mark.parametrize("M,K", [(5, 9225), (5, 12288), (8, 8712), (8, 8720)])
def test_lane_order_with_two_super_chunks_of_8_bit_weights(abq, M, K):
    """The variant with the fewest registers to spare, which exchanges the lanes ahead of the masks: rows of whole vectors, of dwords and
    off dwords, with codes past q bits that the masks have to drop."""
    p, q, N = 8, 7, 70
    c = synth.make_case(p, q, M, N, K, seed=5950 + M, name=f"W{p}A{q} {M}x{N}x{K}")
    print(c.name, flush=True)
    pw = abq.abq_pack_weights(p, to_dev(torch, c.W), to_dev(torch, c.w_scale), to_dev(torch, c.w_zero))
    a = (to_dev(torch, c.A | 0x80), to_dev(torch, c.a_scale), to_dev(torch, c.a_zero))
    out, names = run_named(torch, lambda: abq.abq_gemm_act_codes(p, q, M, N, K, *a, pw, FIELDS, want_acc=True))
    assert len(names) == 1 and "direct_kernel<8, 8, 2, true, true" in names[0], names
    check_against_oracle(c, out[0].cpu().numpy(), out[1].cpu().numpy())
