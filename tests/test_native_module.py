"""The extension module of the online calls, as far as it goes without a device: arguments, errors, threads.  Every call here is one
that is refused: by the module, for want of a stream where there is no device, or by the library (K = 0), which launches nothing."""
import threading
import time

import pytest

from paper_2408_08554_amd import binding as B

torch = pytest.importorskip("torch")

FIELDS = B.ABQ_LAYOUT_FIELDS


def host(*shape, dtype=torch.uint8):
    return torch.zeros(shape, dtype=dtype)


def test_allocations_leave_other_threads_running():
    """A gigabyte of outputs, filled by torch's deterministic mode, takes long enough to see whether another thread stops meanwhile."""
    ticks, stop = [], threading.Event()

    def tick():
        while not stop.is_set():
            ticks.append(time.perf_counter())
            time.sleep(0.002)

    def allocate():
        t0 = time.perf_counter()
        with pytest.raises(RuntimeError):                       # K = 0, and no stream without a device
            B.abq_gemm(4, 8, 1 << 15, 1 << 14, 0, host(16), FIELDS, host(16), FIELDS)
        return t0, time.perf_counter()

    was = torch.are_deterministic_algorithms_enabled()
    torch.use_deterministic_algorithms(True)
    thread = threading.Thread(target=tick)
    try:
        thread.start()
        time.sleep(0.05)
        t0, t1 = allocate()
    finally:
        stop.set()
        thread.join()
        torch.use_deterministic_algorithms(was)
    # (one tick before the allocation and one behind it are possible with the GIL held all the while; freeing holds it)
    inside = [t for t in ticks if t0 < t < t1]
    assert len(inside) >= 6, (len(inside), t1 - t0)


def test_a_failed_allocation_is_an_exception():
    for _ in range(3):
        with pytest.raises(RuntimeError):
            B.abq_gemm(4, 8, 1 << 30, 1 << 30, 0, host(16), FIELDS, host(16), FIELDS)
        with pytest.raises(RuntimeError):
            B.abq_gemm_act_codes(4, 8, 1, -1, 0, host(1, 512), host(1), host(1), host(16), FIELDS)


BEYOND = [1 << 31, -(1 << 31) - 1, (1 << 32) + 8, 1 << 70]


@pytest.mark.parametrize("value", BEYOND)
def test_integers_beyond_32_bits_are_refused(value):
    """Each integer argument in turn; the outputs would otherwise be made, and the problem run, at the size that is left."""
    t, f = host(16), FIELDS
    act = (host(1, 512), host(1), host(1), host(16))
    calls = [lambda *d: B.abq_gemm(*d[:5], t, d[5], t, d[6], host(1)), lambda *d: B.abq_gemm_act_codes(*d[:5], *act, d[5], host(1)),
             lambda *d: B.abq_gemm_act_codes_static(*d[:5], *act, d[5], host(1)), lambda *d: B.abq_f4_gemm(*d[:5], t, t, host(1)),
             lambda *d: B.abq_gemm_act_codes_requant(*d[:5], *act, d[5], d[6], host(1), host(1)),
             lambda *d: B.abq_gemm_grouped(*d[:3], [], d[3], d[4]), lambda *d: B.abq_quant_pack_act(d[0], host(1, 16), d[1]),
             lambda *d: B.abq_pack_act_codes(d[0], host(1, 16), host(1), host(1), d[1]), lambda *d: B.abq_f4_pack_codes(d[0], host(1, 16), host(1), host(1)),
             lambda *d: B.abq_rmsnorm_quant_act(d[0], host(1, 16), host(16), 1e-5), lambda *d: B.abq_silu_mul_quant_act(d[0], host(1, 16), host(1, 16)),
             lambda *d: B.abq_add_rmsnorm_quant_act(d[0], host(1, 16), host(1, 16), host(16), 1e-5)]
    for call, count in zip(calls, (7, 6, 6, 5, 7, 5, 2, 2, 1, 1, 1, 1)):
        for at in range(count):
            args = [2, 2, 1, 64, 0, f, f]
            args[at] = value
            with pytest.raises(OverflowError):
                call(*args)


def test_rows_beyond_32_bits_are_refused():
    wide = host(1).expand(1, (1 << 32) + 16)
    with pytest.raises(OverflowError):
        B.abq_silu_mul_quant_act(8, wide, wide)
    with pytest.raises(OverflowError):
        B.abq_rmsnorm_quant_act(8, wide.T, wide, 1e-5)


def test_integers_of_other_types():
    """What the interpreter takes for an integer, as ctypes does; a float or a text is none."""
    np = pytest.importorskip("numpy")
    for one in (True, np.int64(1), torch.tensor(1)):
        with pytest.raises(RuntimeError):
            B.abq_gemm(4, 8, one, 64, 0, host(16), FIELDS, host(16), FIELDS)
    for other in (1.0, "1", None):
        with pytest.raises(TypeError):
            B.abq_gemm(4, 8, other, 64, 0, host(16), FIELDS, host(16), FIELDS)


def test_operands_that_are_no_tensors():
    """A storage, or any object with a data_ptr() (packed weights: and a device), is an operand; an object without is none, and neither
    is a buffer that make_problems did not make."""
    class Own:
        device = torch.device("cpu")

        def data_ptr(self):
            return 4096

        def numel(self):
            return 1 << 20

    f, storage = FIELDS, host(16).untyped_storage()
    for operand in (storage, Own()):
        for call in (lambda: B.abq_gemm(4, 8, 1, 64, 0, operand, f, operand, f), lambda: B.abq_f4_gemm(2, 2, 1, 64, 0, operand, operand, operand, operand),
                     lambda: B.abq_gemm_act_codes(4, 8, 1, 64, 0, operand, operand, operand, operand, f, operand, operand),
                     lambda: B.abq_gemm_act_codes_static(4, 8, 1, 64, 0, operand, operand, operand, operand, f, operand, operand)):
            with pytest.raises(RuntimeError):                   # (refused no earlier than a tensor)
                call()
    with pytest.raises(RuntimeError):                           # (a workspace says its size too)
        B.abq_gemm(4, 8, 1, 64, 0, Own(), f, Own(), f, Own(), workspace=Own())
    with pytest.raises(AttributeError, match="numel"):
        B.abq_gemm(4, 8, 1, 64, 0, Own(), f, Own(), f, Own(), workspace=storage)
    for other in (7, "text", [host(16)]):
        with pytest.raises((AttributeError, TypeError)):
            B.abq_gemm(4, 8, 1, 64, 0, other, f, host(16), f)
        with pytest.raises((AttributeError, TypeError)):
            B.abq_gemm(4, 8, 1, 64, 0, host(16), f, other, f)
    for other in (bytes(72), bytearray(72), memoryview(bytes(144))):
        with pytest.raises(TypeError):
            B.abq_gemm_grouped(4, 8, 1, other, f, f)


def test_names_of_the_online_calls(monkeypatch):
    """They show in dir() and come with `import *`, as the functions of the module itself do; without a build they are there and raise
    when called."""
    space = {}
    exec("from paper_2408_08554_amd.binding import *", space)
    for name in B._NATIVE:
        assert name in dir(B) and callable(space[name]) and space[name] is getattr(B, name)
    assert {"load", "make_problems", "ABQ_LAYOUT_FIELDS", "AbqError"} <= set(space) and not hasattr(B, "abq_no_such_call")
    for name in B._NATIVE:
        monkeypatch.delattr(B, name)
    for missing in ("LIB_PATH", "NATIVE_PATH"):
        with monkeypatch.context() as m:
            m.setattr(B, missing, "/nonexistent.so")
            m.setattr(B, "_lib", None)
            assert all(hasattr(B, name) for name in B._NATIVE)
            call = B.abq_gemm
            with pytest.raises(RuntimeError, match="is missing"):
                call(4, 8, 1, 64, 0, None, FIELDS, host(16), FIELDS)
    with pytest.raises(RuntimeError) as e:                      # (bound at the call once there is a build)
        call(4, 8, 1, 64, 0, None, FIELDS, host(16), FIELDS, host(1))
    assert "is missing" not in str(e.value)


def test_keywords_and_missing_arguments():
    t, f = host(16), FIELDS
    full = dict(p=4, q=8, M=1, N=64, K=0, packed_act=t, a_layout=f, packed_w=t, w_layout=f, y=host(1))
    with pytest.raises(RuntimeError):                             # (all there: refused by what comes after the arguments)
        B.abq_gemm(**full)
    with pytest.raises(RuntimeError):
        B.abq_gemm(4, 8, 1, 64, 0, t, f, w_layout=f, packed_w=t, workspace=t, want_acc=True, acc=None, y=host(1))
    for name in list(full)[:9]:
        with pytest.raises(TypeError, match="missing required argument: '%s'" % name):
            B.abq_gemm(**{k: v for k, v in full.items() if k != name})
    with pytest.raises(TypeError, match="multiple values for argument 'q'"):
        B.abq_gemm(4, 8, q=8)
    with pytest.raises(TypeError, match="unexpected keyword argument 'z'"):
        B.abq_gemm(**full, z=1)
    with pytest.raises(TypeError, match="at most 13 arguments"):
        B.abq_gemm(*([4] * 14))


def test_checked_tensors_have_to_be_on_the_device():
    row = host(1, 16)
    for call in (lambda: B.abq_quant_pack_act(8, row.half()), lambda: B.abq_pack_act_codes(8, row, host(1, dtype=torch.float32), host(1, dtype=torch.int32)),
                 lambda: B.abq_f4_pack_codes(2, row, host(1, dtype=torch.float32), host(1, dtype=torch.int32)),
                 lambda: B.abq_gemm_act_codes_requant(4, 8, 1, 64, 0, row, row, row, row, FIELDS, 8, host(1, dtype=torch.float32), host(1, dtype=torch.int32))):
        with pytest.raises(AssertionError, match="contiguous device tensor"):
            call()
    with pytest.raises(ValueError, match="two dimensions"):
        B.abq_quant_pack_act(8, host(16))


@pytest.mark.gpu
def test_checked_tensors_have_their_type_and_shape(abq):
    """Refused before anything is launched; the same call with the right tensors goes through."""
    dev = lambda *shape, dtype=torch.uint8: torch.zeros(shape, dtype=dtype, device="cuda")
    codes, scale, zero = dev(2, 64), dev(2, dtype=torch.float32), dev(2, dtype=torch.int32)
    for bad in ((codes.int(), scale, zero), (codes, scale.double(), zero), (codes, scale, zero.long()), (codes, dev(3, dtype=torch.float32), zero),
                (codes, scale, zero.view(2, 1)), (dev(64, 2).T, scale, zero), (codes.cpu(), scale, zero)):
        with pytest.raises(AssertionError, match="contiguous device tensor"):
            abq.abq_pack_act_codes(8, *bad)
    with pytest.raises(B.AbqError) as e:                          # the library's own refusals come with their status
        abq.abq_pack_act_codes(9, codes, scale, zero)
    assert e.value.status == B.ABQ_ERR_BITS
    with pytest.raises(B.AbqError) as e:
        abq.abq_pack_act_codes(8, codes, scale, zero, out=dev(16))
    assert e.value.status == B.ABQ_ERR_SIZE
    given = dev(B.abq_packed_act_bytes(8, 2, 64, FIELDS))
    assert abq.abq_pack_act_codes(8, a_zero=zero, a_codes=codes, a_scale=scale, layout=FIELDS, out=given) is given
