"""The block kernel (prompts over many output tiles): every workgroup shape of every width (tests/test_abi_host.py holds the list against the
library), ragged in all three directions, bit for bit against the tiled
kernel (which writes the int32 accumulator, so a call that asks for it takes that kernel) and against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2408_08554_amd import synth
from helpers import check_against_oracle, check_g128, check_sampled, run_named, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

FIELDS, G128 = 2, 4
WAVES = {"256": "2, 4, 8, ", "192": "2, 4, 4, 3,", "128": "2, 4, 4, 2,", "128x2": "2, 2, 4, 4,", "64x2": "1, 4, 4, 2,"}
# shape by the rule, width, rows, channels, K: fewer steps than the ring has places, parts of a super-chunk, several of them
CASES = [("256", 1, 981, 12680, 518), ("256", 1, 1241, 11606, 106), ("256", 2, 1349, 10535, 103), ("256", 2, 1357, 10440, 1030), ("256", 3, 1223, 9940, 1100),
         ("256", 4, 1157, 10048, 520), ("256", 5, 900, 12816, 101), ("256", 6, 960, 12385, 530), ("256", 7, 654, 12064, 1040), ("256", 8, 846, 9375, 1027),
         ("192", 1, 629, 9736, 185), ("192", 1, 632, 9770, 530), ("192", 2, 626, 6696, 106), ("192", 2, 1361, 4356, 568), ("192", 3, 1345, 4384, 106),
         ("192", 4, 257, 13216, 528), ("192", 5, 260, 13117, 536), ("192", 5, 260, 13496, 1044), ("192", 6, 261, 13168, 521), ("192", 7, 386, 12224, 108),
         ("192", 8, 261, 13176, 520), ("128", 4, 134, 10912, 1061), ("128", 5, 132, 11051, 1630), ("128", 6, 132, 11069, 1028), ("128", 6, 193, 12856, 1589),
         ("128", 7, 133, 12304, 1029), ("128", 8, 130, 11038, 520), ("128x2", 1, 396, 13981, 107), ("128x2", 2, 513, 12296, 110),
         ("128x2", 2, 1129, 5411, 100), ("128x2", 3, 579, 10006, 101), ("128x2", 3, 1164, 5128, 515), ("128x2", 4, 394, 9581, 100),
         ("128x2", 5, 328, 10910, 101), ("128x2", 6, 258, 13288, 104), ("128x2", 7, 389, 12832, 103), ("128x2", 8, 468, 8202, 100),
         ("64x2", 1, 71, 8462, 1106), ("64x2", 2, 67, 4631, 103), ("64x2", 2, 194, 12504, 1040), ("64x2", 3, 259, 9904, 101), ("64x2", 4, 264, 11080, 100),
         ("64x2", 5, 194, 12208, 103), ("64x2", 6, 201, 12192, 101), ("64x2", 7, 133, 12456, 101), ("64x2", 8, 65, 8304, 563),
         ("64x2", 4, 1000, 1100, 33000)]   # (sums past 2^23: the 32-bit epilogue)


def problem(abq, shape, p, q, M, N, K):
    c = synth.make_case(p, q, M, N, K, seed=7300 + 10 * p + q, name=f"block {shape} W{p}A{q} {M}x{N}x{K}")
    print(c.name, flush=True)
    c.W[::5], c.A[::7] = (1 << p) - 1, (1 << q) - 1   # the largest codes, whole rows of them, against each other
    pw = abq.abq_pack_weights(p, to_dev(torch, c.W), to_dev(torch, c.w_scale), to_dev(torch, c.w_zero))
    return c, pw, abq.abq_pack_act_codes(q, to_dev(torch, c.A), to_dev(torch, c.a_scale), to_dev(torch, c.a_zero))


@pytest.mark.parametrize("q", [8, 4])
@pytest.mark.parametrize("shape,p,M,N,K", CASES)
def test_block_equals_the_tiled_kernel(abq, shape, p, q, M, N, K):
    c, pw, pa = problem(abq, shape, p, q, M, N, K)
    (y0, acc0), names = run_named(torch, lambda: abq.abq_gemm(p, q, M, N, K, pa, FIELDS, pw, FIELDS, want_acc=True))
    assert len(names) == 1 and f"tiled_kernel<{p}, " in names[0], names
    (y, _), names = run_named(torch, lambda: abq.abq_gemm(p, q, M, N, K, pa, FIELDS, pw, FIELDS))
    assert len(names) == 1 and f"block_kernel<{p}, {WAVES[shape]}" in names[0], names
    assert torch.equal(y.view(torch.int16), y0.view(torch.int16))
    check_sampled(c, y.cpu().numpy(), acc0.cpu().numpy())


@pytest.mark.parametrize("shape,p,M,N,K", [c for c in CASES if c[1] in (4, 7, 8) and c[4] < 2000])
def test_block_writes_the_next_layers_codes(abq, shape, p, M, N, K):
    """Output codes with and without the binary16 output: those of the values that it stores."""
    q, qo = 8, 6
    c, pw, pa = problem(abq, shape, p, q, M, N, K)
    y0, _ = abq.abq_gemm(p, q, M, N, K, pa, FIELDS, pw, FIELDS)
    a, sa, za = to_dev(torch, c.A), to_dev(torch, c.a_scale), to_dev(torch, c.a_zero)
    rng = np.random.default_rng(5)
    so, zo = rng.uniform(0.5, 4.0, M).astype(np.float32), rng.integers(0, 1 << qo, M).astype(np.int32)
    dso, dzo = to_dev(torch, so), to_dev(torch, zo)
    call = lambda **kw: abq.abq_gemm_act_codes_requant(p, q, M, N, K, a, sa, za, pw, FIELDS, qo, dso, dzo, **kw)
    (codes, y), names = run_named(torch, call)
    assert f"block_kernel<{p}, {WAVES[shape]}" in names[-1], names
    assert torch.equal(y.view(torch.int16), y0.view(torch.int16))
    assert np.array_equal(codes.cpu().numpy(), oracle.requant(y0.cpu().numpy(), qo, so, zo))
    assert torch.equal(call(want_y=False)[0], codes)


@pytest.mark.parametrize("shape,p,M,N,K", [c for c in CASES if not (c[1] in (4, 7, 8) and c[4] < 2000)])
def test_block_codes_of_the_other_widths(abq, shape, p, M, N, K):
    """The same for every other width and for sums past 2^23, with parameters that clamp codes at both ends."""
    q, qo = 5 if p % 2 else 8, 8 if p % 2 else 3
    c, pw, _ = problem(abq, shape, p, q, M, N, K)
    a, sa, za = to_dev(torch, c.A), to_dev(torch, c.a_scale), to_dev(torch, c.a_zero)
    y0, _ = abq.abq_gemm_act_codes(p, q, M, N, K, a, sa, za, pw, FIELDS)
    rng = np.random.default_rng(6)
    spread = np.maximum(np.abs(y0.float().cpu().numpy()).max(axis=1), 1e-3)
    so = (spread / (1 << qo) * rng.choice([0.5, 2.0, 4.0], M)).astype(np.float32)
    zo = rng.integers(-3, (1 << qo) + 3, M).astype(np.int32)
    dso, dzo = to_dev(torch, so), to_dev(torch, zo)
    call = lambda **kw: abq.abq_gemm_act_codes_requant(p, q, M, N, K, a, sa, za, pw, FIELDS, qo, dso, dzo, **kw)
    codes, y = call()
    (only, _), names = run_named(torch, lambda: call(want_y=False))
    assert f"block_kernel<{p}, {WAVES[shape]}" in names[-1], names
    assert torch.equal(y.view(torch.int16), y0.view(torch.int16))
    assert np.array_equal(codes.cpu().numpy(), oracle.requant(y0.cpu().numpy(), qo, so, zo))
    assert torch.equal(only, codes)


# what the rule leaves to the tiled kernel: width, rows, channels, K, and the tile (channels of W per wave / 16, rows of A / 16)
DECLINED = [(1, 67, 4512, 113, "1, 4"), (1, 74, 4140, 2535, "1, 4"), (1, 387, 12760, 1048, "2, 4"), (2, 68, 4864, 103, "1, 4"), (2, 68, 4654, 1687, "1, 4"),
            (2, 388, 12376, 514, "2, 4"), (2, 1191, 13376, 1552, "4, 4"), (3, 68, 4097, 536, "1, 4"), (3, 1269, 4808, 535, "2, 4"), (4, 65, 4528, 100, "1, 4"),
            (4, 69, 4977, 2647, "1, 4"), (4, 776, 10280, 101, "2, 4"), (5, 68, 4273, 1359, "1, 4"), (5, 728, 10888, 100, "2, 4"), (6, 65, 4469, 533, "1, 4"),
            (6, 587, 13240, 100, "2, 4"), (6, 1386, 13592, 1034, "2, 8"), (7, 73, 4759, 568, "1, 4"), (7, 1181, 4816, 528, "2, 4"), (7, 450, 12384, 1583, "2, 8"),
            (8, 75, 4320, 104, "1, 4"), (8, 73, 4129, 1172, "1, 4")]


@pytest.mark.parametrize("q", [8, 3])
@pytest.mark.parametrize("p,M,N,K,tile", DECLINED)
def test_tiled_kernel_by_the_rule_without_accumulator(abq, p, q, M, N, K, tile):
    """Ordinary calls that the block kernel leaves alone run the tiled kernel's epilogue without accumulator; calls that ask for it, the other one."""
    c, pw, pa = problem(abq, "declined", p, q, M, N, K)
    call = lambda **kw: abq.abq_gemm(p, q, M, N, K, pa, FIELDS, pw, FIELDS, **kw)
    (y, none), names = run_named(torch, call)
    assert none is None and len(names) == 1 and f"tiled_kernel<{p}, {tile}, " in names[0], names
    y0, acc0 = call(want_acc=True)
    assert torch.equal(y.view(torch.int16), y0.view(torch.int16))
    check_sampled(c, y.cpu().numpy(), acc0.cpu().numpy())


@pytest.mark.parametrize("mt,ntw,wd", [(4, 1, 2), (4, 1, 4), (4, 2, 2), (4, 2, 4), (4, 4, 2), (8, 1, 2), (8, 2, 2), (8, 4, 2)])
@pytest.mark.parametrize("p,q", [(1, 8), (2, 3), (3, 8), (4, 4), (5, 8), (6, 6), (7, 8), (8, 8)])
def test_tiled_shapes_by_plan_entry_without_accumulator(abq, p, q, mt, ntw, wd):
    """Every tile and ring depth through the epilogue of an ordinary call, against the one that writes the accumulator as well."""
    if wd == 4 and ntw == 2 and p >= 7:
        pytest.skip("no deep ring with two tiles of 7 or 8 bits per wave")
    for M, N, K in [(65, 40, 200), (200, 330, 1100), (130, 72, 3590)]:
        c, pw, pa = problem(abq, f"tile {mt} {ntw} {wd}", p, q, M, N, K)
        call = lambda **kw: abq.abq_gemm(p, q, M, N, K, pa, FIELDS, pw, FIELDS, **kw)
        abq.abq_plan_set(p, q, M, N, K, tiled_mt=mt, tiled_ntw=ntw, tiled_wd=wd)
        try:
            (y, _), names = run_named(torch, call)
            y0, acc0 = call(want_acc=True)
        finally:
            abq.abq_plan_set(p, q, M, N, K)
        assert len(names) == 1 and f"tiled_kernel<{p}, {ntw}, {mt}, {wd}>" in names[0], names
        assert torch.equal(y.view(torch.int16), y0.view(torch.int16))
        check_against_oracle(c, y.cpu().numpy(), acc0.cpu().numpy())


@pytest.mark.parametrize("plan,kernel", [(dict(tiled_mt=4), "tiled_kernel"), (dict(tiled_ntw=2), "tiled_kernel"), (dict(tiled_wd=2), "tiled_kernel"),
                                         (dict(tiled_band=2), "tiled_kernel"), (dict(skinny_waves=4), "block_kernel"), (dict(skinny_kgroups=2), "block_kernel"),
                                         (dict(direct_r=1), "block_kernel")])
def test_tiled_knobs_keep_the_tiled_kernel(abq, plan, kernel):
    """As the header says: any knob of the tiled kernel takes a problem from the block kernel, the decode kernels' knobs do not."""
    p, q, M, N, K = 4, 8, 264, 11080, 100
    c, pw, pa = problem(abq, "64x2", p, q, M, N, K)
    call = lambda: abq.abq_gemm(p, q, M, N, K, pa, FIELDS, pw, FIELDS)[0]
    y0, names = run_named(torch, call)
    assert "block_kernel" in names[-1], names
    abq.abq_plan_set(p, q, M, N, K, **plan)
    try:
        y, names = run_named(torch, call)
    finally:
        abq.abq_plan_set(p, q, M, N, K)
    assert len(names) == 1 and kernel in names[0], names
    assert torch.equal(y.view(torch.int16), y0.view(torch.int16))


def test_tuner_checks_the_call_that_it_times(abq):
    """Its timed call runs the block kernel by the rule; the accumulator comes from another kernel, so one call cannot stand for both."""
    from paper_2408_08554_amd import tune
    prob = tune.Problem(4, 8, 264, 11080, 100, rotate_bytes=1 << 22, launches=4)
    assert "block_kernel" in run_named(torch, lambda: prob.call(0))[1][-1]
    assert "tiled_kernel" in run_named(torch, lambda: prob.call(0, acc=prob.acc))[1][-1]
    asked, call = [], prob.call
    prob.call = lambda i, acc=None: (asked.append(acc is not None), call(i, acc=acc))
    out = prob.result()
    assert sorted(asked) == [False, True] and len(out) == 3 and torch.equal(out[0], out[1])


# both shapes by the rule, widths of one and of two plane groups, a last group that is short and groups past K, ragged rows and channels
G128_CASES = [("2, 4, 8,", 1, 577, 10147, 1539), ("2, 4, 8,", 2, 454, 12312, 1547), ("2, 4, 8,", 3, 322, 11195, 1544),
              ("2, 4, 8,", 4, 580, 9735, 1561), ("2, 4, 8,", 5, 391, 9408, 1541), ("2, 4, 8,", 6, 331, 11022, 1665),
              ("1, 4, 8,", 1, 195, 12184, 1652), ("1, 4, 8,", 2, 196, 12712, 1579), ("1, 4, 8,", 3, 193, 12280, 1546),
              ("1, 4, 8,", 4, 194, 12499, 1597), ("1, 4, 8,", 5, 202, 12293, 2049), ("1, 4, 8,", 6, 193, 12752, 1556)]


@pytest.mark.parametrize("waves,p,M,N,K", G128_CASES)
@pytest.mark.parametrize("q", [8, 5])
def test_block_per_group_weights(abq, waves, p, q, M, N, K):
    """Zero-points and codes at both ends of their ranges against each other.  The groups are summed in the tiled per-group kernel's order, so
    every row has the bits that it has in a call of 64 rows, which that kernel takes; some rows against the oracle."""
    c = synth.make_case(p, q, M, N, K, seed=7500 + 10 * p + q, name=f"block g128 W{p}A{q} {M}x{N}x{K}")
    print(c.name, flush=True)
    sh, zg = synth.group_quant_params(c)
    top, atop = (1 << p) - 1, (1 << q) - 1
    zg[:, 0::3], zg[:, 1::3] = 0, top
    c.W[0::3], c.W[1::3] = top, 0
    c.A[0::4], c.A[1::4] = atop, 0
    c.a_zero[0::2], c.a_zero[1::2] = 0, atop
    c.a_scale[:] = np.float32(1e-4)
    pw = abq.abq_pack_weights_g128(p, to_dev(torch, c.W), to_dev(torch, sh.view(np.float16)), to_dev(torch, zg))
    A, sa, za = to_dev(torch, c.A), to_dev(torch, c.a_scale), to_dev(torch, c.a_zero)
    pa = abq.abq_pack_act_codes(q, A, sa, za)
    (y, _), names = run_named(torch, lambda: abq.abq_gemm(p, q, M, N, K, pa, FIELDS, pw, G128))
    assert len(names) == 1 and f"block_g128_kernel<{p}, {waves}" in names[0], names
    for m in range(0, M, 64):
        rows = min(64, M - m)
        if rows < 33:
            m, rows = M - 64, 64
        part = abq.abq_pack_act_codes(q, A[m:m + rows].clone(), sa[m:m + rows].clone(), za[m:m + rows].clone())
        call = lambda: abq.abq_gemm(p, q, rows, N, K, part, FIELDS, pw, G128)
        (ref, _), names = run_named(torch, call) if m == 0 else (call(), ["tiled_g128_kernel"])
        assert "tiled_g128_kernel" in names[0], names
        assert torch.equal(y[m:m + rows].view(torch.int16), ref.view(torch.int16))
    ms = np.r_[0:8, M - 8:M]
    sub = synth.Case(p, q, len(ms), N, K, c.W, c.A[ms], c.w_scale, c.w_zero, c.a_scale[ms], c.a_zero[ms], c.seed, c.name)
    check_g128(sub, sh, zg, y.cpu().numpy()[ms])
