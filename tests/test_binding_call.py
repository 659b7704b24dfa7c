"""The native half of the binding's product call: what it refuses and what it leaves to ctypes (before any HIP call, on CPU
tensors), and that the index list and the views are those of the workspace whatever form that has."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2604_02525_amd import binding as ah


class Renamed(ah.Operand):
    """An operand that is not exactly the binding's type: described by its c()."""


def cpu_call(cls=ah.Operand, block=32, nbytes=1 << 20, strategy=ah.ADAHOP_IHT, k=0, **kw):
    x = cls(torch.zeros(64, 64, dtype=torch.bfloat16), True)
    return ah.adahop_gemm(x, x, strategy, block, k, Cout=torch.zeros(64, 64), workspace=torch.zeros(nbytes, dtype=torch.uint8),
                          stream=0, **kw)


@pytest.mark.parametrize("cls", [ah.Operand, Renamed])
def test_refused_calls_raise_as_the_entry_point_says(cls):
    with pytest.raises(ah.AdahopError, match="adahop_gemm: .*argument") as e:
        cpu_call(cls, block=33)
    assert e.value.status == ah.ADAHOP_E_INVALID_ARG
    with pytest.raises(ah.AdahopError, match="adahop_gemm: ") as e:
        cpu_call(cls, nbytes=64)
    assert e.value.status == ah.ADAHOP_E_WORKSPACE
    with pytest.raises(ah.AdahopError, match="adahop_gemm_ex: "):
        cpu_call(cls, block=33, sr_seed_a=5)
    with pytest.raises(C.ArgumentError):
        cpu_call(cls, block=32.0)
    with pytest.raises(AttributeError):
        cpu_call(cls, strategy=ah.ADAHOP_IHT_OE_K, k=3, block=33, idx=[1, 2, 3])


class Index:
    def __init__(self, value):
        self.value = value

    def __index__(self):
        return self.value


class AsParameter:
    def __init__(self, value):
        self._as_parameter_ = value


class Buffer:
    """No torch tensor, but all that the binding asks of one."""

    def __init__(self, t):
        self.t, self.device, self.shape = t, t.device, t.shape

    def __getattr__(self, name):
        if name in ("data_ptr", "dim", "stride", "element_size", "numel"):
            return getattr(self.t, name)
        raise AttributeError(name)


INTEGERS = [int, np.int64, np.int32, np.uint8, Index, AsParameter, C.c_int]


@pytest.mark.parametrize("integer", INTEGERS)
def test_integers_are_what_ctypes_takes(integer):
    with pytest.raises(ah.AdahopError) as e:            # the entry point was reached, and refused the block
        cpu_call(block=integer(33))
    assert e.value.status == ah.ADAHOP_E_INVALID_ARG
    with pytest.raises(ah.AdahopError) as e:            # every argument accepted up to the workspace
        cpu_call(block=integer(32), strategy=integer(ah.ADAHOP_IHT), nbytes=64)
    assert e.value.status == ah.ADAHOP_E_WORKSPACE
    for refused in (33.0, "33", None, C.c_long(33)):
        with pytest.raises(C.ArgumentError):
            cpu_call(block=refused)


@pytest.mark.parametrize("count", [int, np.int64])
def test_objects_with_a_data_pointer(count):
    def buffer_op(t, kc):
        return ah.Operand(Buffer(t), kc)
    for strategy, k in ((ah.ADAHOP_IHT, 0), (ah.ADAHOP_IHT_OE_ROW, 3)):
        for cls in (buffer_op, ah.Operand):
            with pytest.raises(ah.AdahopError) as e:
                cpu_call(cls, block=33, strategy=strategy, k=count(k))
            assert e.value.status == ah.ADAHOP_E_INVALID_ARG
            with pytest.raises(ah.AdahopError) as e:
                cpu_call(cls, nbytes=64, strategy=strategy, k=count(k), idx=Buffer(torch.zeros(8, dtype=torch.int32)))
            assert e.value.status == ah.ADAHOP_E_WORKSPACE


@pytest.mark.gpu
@pytest.mark.parametrize("strategy,k", [(ah.ADAHOP_IHT, 0), (ah.ADAHOP_IHT_OE_ROW, 3), (ah.ADAHOP_IHT_OE_COL, 5), (ah.ADAHOP_IHT_OE_K, 7)])
def test_index_list_and_views_in_every_form_of_the_workspace(strategy, k):
    gen = torch.Generator(device="cuda").manual_seed(9)
    M, N, K = 96, 160, 320
    x = torch.randn(M, K, generator=gen, device="cuda").to(torch.bfloat16)
    w = torch.randn(N, K, generator=gen, device="cuda").to(torch.bfloat16)
    need = ah.adahop_gemm_workspace_bytes(M, N, K, strategy, k)
    flat = torch.empty(need + 512, dtype=torch.uint8, device="cuda")
    spaces = [None, flat[:need], flat[256:256 + need], flat[:need // 256 * 256 + 256].view(-1, 256).view(-1)]
    want = None
    for cls in (ah.Operand, Renamed):
        for ws in spaces:
            r = ah.adahop_gemm(cls(x, True), cls(w, True), strategy, 64, k, workspace=ws)
            torch.cuda.synchronize()
            assert r["idx"].dtype == torch.int32 and r["idx"].shape == (k,) and r["idx"].is_cuda
            space, L = r["workspace"], r["layout"]
            dim = {ah.ADAHOP_IHT_OE_ROW: M, ah.ADAHOP_IHT_OE_COL: N, ah.ADAHOP_IHT_OE_K: K}.get(strategy, 0)
            for name, shape in (("a_codes", (M, K // 2)), ("a_scales", (M, K // 32)), ("b_codes", (N, K // 2)), ("b_scales", (N, K // 32)),
                                ("mask", (dim,))):
                v = r[name]
                assert v.shape == shape and v.dtype == torch.uint8 and v.is_contiguous()
                if dim or name != "mask":
                    assert v.data_ptr() == space.data_ptr() + getattr(L, name)
            got = {n: r[n].clone() for n in ("C", "idx", "a_codes", "a_scales", "b_codes", "b_scales", "mask")}
            if want is None:
                want = got
            for n in got:
                assert torch.equal(got[n], want[n]), n
    for integer in INTEGERS:
        count = integer if integer in (int, np.int64) else int
        r = ah.adahop_gemm(ah.Operand(x, True), ah.Operand(Buffer(w), True), count(strategy), integer(64), count(k),
                           workspace=flat[:need],
                           stream=C.c_void_p(torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
        for n in ("C", "idx", "a_codes", "a_scales", "b_codes", "b_scales"):
            assert torch.equal(r[n], want[n]), n
    if k:
        again = ah.adahop_gemm(ah.Operand(x, True), ah.Operand(w, True), strategy, 64, k, idx=want["idx"])
        torch.cuda.synchronize()
        assert torch.equal(again["C"], want["C"]) and torch.equal(again["idx"], want["idx"])
