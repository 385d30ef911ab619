"""The C-ABI library loads, exports every symbol the header declares, and rejects bad
arguments on the host before anything is launched (so these run without a GPU)."""
import ctypes as C
import os
import re
import threading
import time

import numpy as np
import pytest
import torch

import paper_2009_08065_amd as bsp

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_symbols():
    text = open(os.path.join(ROOT, "include", "bsp.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(bsp_[a-z_0-9]+)\s*\(", text)))


def test_every_declared_symbol_is_exported():
    L = bsp.lib()
    names = declared_symbols()
    assert {"bsp_group_norms", "bsp_penalty_grad", "bsp_prune_mask", "bsp_pack_count", "bsp_pack", "bsp_linear",
            "bsp_packed_validate", "bsp_compression_rate", "bsp_status_string"} <= set(names)
    for n in names:
        assert hasattr(L, n), n


def test_status_strings_and_rate():
    L = bsp.lib()
    assert L.bsp_status_string(0) == b"ok"
    assert all(L.bsp_status_string(i) for i in range(8))
    assert bsp.bsp_compression_rate(768, 768, 16, 48 * 384) == 2.0
    assert abs(bsp.bsp_compression_rate(100, 100, 10, 700) - 1 / 0.7) < 1e-12   # Sec. 4.4: 30 % sparsity
    assert bsp.bsp_compression_rate(8, 8, 4, 0) == float("inf")


def test_host_side_argument_checks():
    L = bsp.lib()
    one = C.c_void_p(16)   # never dereferenced: every call below fails validation first
    OK, NULL, SHAPE, DTYPE, CAP = 0, 1, 2, 3, 4
    assert L.bsp_group_norms(None, 0, 16, 8, 16, 1e-6, 0, one, one, one, None) == NULL
    assert L.bsp_group_norms(one, 0, 17, 8, 16, 1e-6, 0, one, one, one, None) == SHAPE      # M % R
    assert L.bsp_group_norms(one, 0, 16, 8, 0, 1e-6, 0, one, one, one, None) == SHAPE       # R < 1
    assert L.bsp_group_norms(one, 0, 130, 8, 65, 1e-6, 0, one, one, one, None) == SHAPE     # R > 64
    assert L.bsp_group_norms(one, 7, 16, 8, 16, 1e-6, 0, one, one, one, None) == DTYPE
    assert L.bsp_group_norms(one, 0, 16, 8, 16, 1e-6, 5, one, one, one, None) == DTYPE
    assert L.bsp_group_norms(one, 0, 16, 8, 16, 1e-6, 0, None, None, None, None) == OK      # nothing to do
    assert L.bsp_penalty_grad(one, 0, 16, 8, 16, None, 0.1, 0, 0, one, None, None, 0, None) == NULL
    assert L.bsp_penalty_grad(one, 0, 16, 8, 16, one, 0.1, 0, 0, one, one, one, 0, None) == CAP
    assert L.bsp_prune_mask(None, 1, 8, 0.0, -1, 0, one, None, None, 0, None) == NULL
    assert L.bsp_prune_mask(one, 0, 8, 0.0, -1, 0, one, None, None, 0, None) == SHAPE
    assert L.bsp_prune_mask(one, 1 << 20, 1 << 20, 0.0, -1, 0, one, None, None, 0, None) == SHAPE
    assert L.bsp_prune_mask(one, 2, 8, 0.0, 3, 1, one, None, one, 4, None) == CAP
    assert L.bsp_prune_mask(one, 2, 8, 0.0, 3, 9, one, None, one, 1 << 20, None) == DTYPE
    assert L.bsp_prune_mask_static(one, 1 << 20, 1 << 20, 0.0, 5, 1, one, None, None) == SHAPE   # beyond its scratch
    assert L.bsp_prune_mask_count(one, 2, 8, 0.0, 3, 1, one, None, 32, None, one, one, 1 << 20, None) == NULL
    assert L.bsp_prune_mask_count(one, 2, 8, 0.0, 3, 1, one, None, 5, one, one, one, 1 << 20, None) == SHAPE
    assert L.bsp_prune_mask_count(one, 2, 8, 0.0, 3, 1, one, None, 32, one, one, one, 4, None) == CAP
    assert L.bsp_prune_mask_count(one, 2, 8, 0.0, 3, 1, one, None, 32, one, one, None, 0, None) == NULL
    assert L.bsp_prune_mask_static(one, 0, 8, 0.0, -1, 0, one, None, None) == SHAPE
    assert L.bsp_pack_count(one, 2, 8, 3, one, one, None) == SHAPE                           # k_align
    assert L.bsp_pack_count(None, 2, 8, 16, one, one, None) == NULL
    assert L.bsp_pack(one, 0, 16, 8, 16, one, 16, one, one, -1, one, one, 0, None) == CAP
    assert L.bsp_pack(one, 0, 16, 8, 16, one, 16, one, one, 0, None, None, 0, None) == OK    # empty storage
    assert L.bsp_pack(one, 0, 16, 8, 16, one, 16, one, one, 5, None, one, 0, None) == NULL
    assert L.bsp_pack(one, 0, 16, 8, 16, one, 16, one, one, 5, one, one, 9, None) == DTYPE
    assert L.bsp_linear(None, 1, 4, 16, 8, 16, 32, one, one, one, one, None, one, None) == NULL
    assert L.bsp_linear(one, 1, 4, 24, 8, 16, 32, one, one, one, one, None, one, None) == SHAPE
    assert L.bsp_linear(one, 1, 0, 16, 8, 16, 32, one, one, one, one, None, one, None) == OK  # no tokens
    assert L.bsp_linear(C.c_void_p(8), 1, 4, 16, 8, 16, 32, one, one, one, one, None, one, None) == SHAPE  # alignment
    assert L.bsp_linear(one, 5, 4, 16, 8, 16, 32, one, one, one, one, None, one, None) == DTYPE
    assert L.bsp_linear_transposed(None, 1, 4, 16, 8, 16, 32, one, one, one, one, None, one, None) == NULL
    assert L.bsp_linear_transposed(one, 1, 4, 24, 8, 16, 32, one, one, one, one, None, one, None) == SHAPE
    assert L.bsp_linear_transposed(one, 1, 4, 16, 70000, 16, 32, one, one, one, one, None, one, None) == SHAPE
    assert L.bsp_linear_transposed(one, 1, 0, 16, 8, 16, 32, one, one, one, one, None, one, None) == OK  # no tokens
    assert L.bsp_linear_transposed(one, 7, 4, 16, 8, 16, 32, one, one, one, one, None, one, None) == DTYPE
    assert L.bsp_linear_transposed_dense(None, 1, 4, 16, 8, one, None, one, None) == NULL
    assert L.bsp_linear_transposed_dense(one, 9, 4, 16, 8, one, None, one, None) == DTYPE
    assert L.bsp_linear_transposed_dense(one, 1, 4, 0, 8, one, None, one, None) == SHAPE
    assert L.bsp_linear_transposed_dense(one, 1, 0, 16, 8, one, None, one, None) == OK       # no tokens
    # (X, dY, xdt, T, M, N, R, k_align, blk_cnt, blk_ptr, col_idx, capacity_cols, D, gdt, ws, ws_bytes, stream)
    assert L.bsp_linear_dvals(one, one, 1, 4, 16, 8, 16, 32, None, one, one, 32, one, 1, None, 0, 0, None) == NULL
    assert L.bsp_linear_dvals(one, one, 1, 4, 24, 8, 16, 32, one, one, one, 32, one, 1, None, 0, 0, None) == SHAPE  # M % R
    assert L.bsp_linear_dvals(one, one, 1, 4, 16, 8, 16, 5, one, one, one, 32, one, 1, None, 0, 0, None) == SHAPE   # k_align
    assert L.bsp_linear_dvals(one, one, 7, 4, 16, 8, 16, 32, one, one, one, 32, one, 1, None, 0, 0, None) == DTYPE
    assert L.bsp_linear_dvals(one, one, 1, 4, 16, 8, 16, 32, one, one, one, 32, one, 9, None, 0, 0, None) == DTYPE
    assert L.bsp_linear_dvals(one, one, 1, 4, 16, 8, 16, 32, one, one, None, 0, None, 1, None, 0, 0, None) == OK    # nothing kept
    assert L.bsp_linear_dvals(one, one, 1, 4, 16, 8, 16, 32, one, one, one, 32, None, 1, None, 0, 0, None) == NULL  # no D
    ws = C.c_void_p(4096)
    assert L.bsp_linear_dvals(C.c_void_p(64), C.c_void_p(64), 1, 4, 16, 8, 16, 32, one, one, one, 32, one, 1, ws, 16, 0, None) == CAP
    assert L.bsp_linear_dvals(one, one, 1, 4, 16, 8, 16, 32, one, one, one, 32, one, 1, None, 0, 5, None) == SHAPE  # ws_state
    assert L.bsp_linear_dvals_workspace_bytes(3072, 1024, 16, 45000) > 256 * 12 * 4096 * 4      # 256 units of partial sums
    assert L.bsp_linear_dvals_workspace_bytes(3072, 1024, 5, 45000) == 0                         # M % R
    assert L.bsp_packed_validate(16, 8, 16, 16, None, one, one, 0, one, None) == NULL
    assert L.bsp_penalty_grad_workspace_bytes(32, 300, 16) == 2 * 2 * 8
    assert L.bsp_prune_mask_workspace_bytes(4, 100, 1) >= 2 * (2048 + 64) * 4   # two histogram slots at least
    assert L.bsp_prune_mask_workspace_bytes(256, 4096, 1) > L.bsp_prune_mask_workspace_bytes(4, 100, 1)
    assert L.bsp_prune_mask_workspace_bytes(4, 100, 0) == 0


def test_expansion_is_not_offered_beyond_its_grid():
    """More columns than the expansion's grid has rows for: no scratch, so the transposed product stays with the kernel on the storage."""
    L = bsp.lib()
    cols = 65535 * 256
    assert L.bsp_linear_transposed_workspace_bytes(bsp.BF16, 4, 64, cols, 16) >= 2 * 64 * cols
    assert L.bsp_linear_transposed_workspace_bytes(bsp.BF16, 4, 64, cols + 1, 16) == 0
    assert L.bsp_linear_transposed_workspace_bytes(bsp.BF16, 4, 64, 1 << 32, 16) == 0


def test_linear_sized_refuses_a_negative_count():
    one = C.c_void_p(16)
    assert bsp.lib().bsp_linear_sized(one, 0, 4, 64, 64, 16, 32, one, one, one, one, -1, None, one, None, 0, None) == 4
    assert bsp.lib().bsp_linear_sized(None, 0, 4, 64, 64, 16, 32, one, one, one, one, 64, None, one, None, 0, None) == 1
    assert bsp.lib().bsp_linear_sized(one, 0, 0, 64, 64, 16, 32, one, one, one, one, 64, None, one, None, 0, None) == 0   # no tokens


def test_expansion_pays_for_enough_tokens_only():
    """The layer's scratch query: calls whose expansion alone costs more than the gather get none (all three were measured 2 to 5
    times slower with it), calls of many tokens of layers that keep much get some."""
    L = bsp.lib()
    q = L.bsp_linear_workspace_bytes
    kept = lambda M, N, R, rate: int(M // R * N / rate) // 32 * 32
    for M, N, R, rate, T in ((30528, 768, 8, 1.1, 1), (30528, 768, 8, 1.1, 40), (4096, 1024, 1, 1.43, 40), (16384, 4096, 16, 1.1, 40),
                             (16384, 4096, 4, 1.43, 1), (2048, 2048, 1, 1.43, 40)):
        assert q(bsp.BF16, T, M, N, R, 32, kept(M, N, R, rate)) == 0, (M, N, R, rate, T)
    for M, N, R, rate, T in ((1024, 4096, 16, 1.43, 8192), (1024, 4096, 16, 5.0, 8192), (768, 3072, 8, 2.0, 4096), (4096, 1024, 16, 1.43, 8192),
                             (4096, 1024, 1, 1.43, 1100)):
        assert q(bsp.BF16, T, M, N, R, 32, kept(M, N, R, rate)) > 0, (M, N, R, rate, T)


def test_expansion_and_the_rounds_of_the_gather():
    """Calls of whole rounds of the gather's workgroups stay with it (measured 1.1 to 1.9 times slower by the expansion), calls of a few
    tokens more do not; and the rule has no end at 8192 tokens or 16384 rows (the gather takes 1.2 to 3 times as long as the expansion there)."""
    q = bsp.lib().bsp_linear_workspace_bytes
    kept = lambda M, N, R, rate: int(M // R * N / rate) // 32 * 32
    for M, N, R, rate, T in ((768, 768, 16, 3.0, 8192), (1024, 1024, 16, 3.0, 8192), (896, 896, 16, 3.0, 8147), (512, 2048, 16, 5.0, 4080),
                             (18096, 2944, 2, 1.3, 33)):
        assert q(bsp.BF16, T, M, N, R, 32, kept(M, N, R, rate)) == 0, (M, N, R, rate, T)
    for M, N, R, rate, T in ((1024, 4096, 16, 5.0, 2100), (20000, 512, 16, 2.0, 3000)):
        assert q(bsp.BF16, T, M, N, R, 32, kept(M, N, R, rate)) > 0, (M, N, R, rate, T)
    for M, N, R, rate in ((768, 768, 8, 2.0), (1024, 1024, 32, 1.5), (4096, 1024, 8, 2.0), (640, 2560, 32, 3.0)):
        for T in (8192, 8193, 9000, 40000):
            assert q(bsp.F16, T, M, N, R, 32, kept(M, N, R, rate)) > 0, (M, N, R, rate, T)


class _Elsewhere:
    """What the binding asks of an object that is no plain tensor."""
    is_cuda = True

    def __init__(self, dtype=torch.float32, dense=True, at=4096):
        self.dtype, self.dense, self.at = dtype, dense, at

    def is_contiguous(self):
        return self.dense

    def data_ptr(self):
        return self.at


def test_native_functions_check_what_they_are_given():
    """The native functions refuse what the binding refused: tensors that are not on the GPU or not contiguous, of another
    type than the function's where that is checked, numbers in the place of tensors and the other way round."""
    n = bsp.bsp._native()
    host = torch.zeros(4, 4)
    with pytest.raises(ValueError, match="contiguous GPU tensor"):
        n.bsp_mask_weights(host, 0, 4, 4, 2, None, 0)
    with pytest.raises(ValueError, match="contiguous GPU tensor"):
        n.bsp_mask_weights(_Elsewhere(dense=False), 0, 4, 4, 2, None, 0)
    with pytest.raises(ValueError, match="expected dtype torch.uint8, got torch.float32"):
        n.bsp_mask_weights(_Elsewhere(), 0, 4, 4, 2, _Elsewhere(), 0)
    for args in ((4096, 0, 4, 4, 2, None, 0), (None, host, 4, 4, 2, None, 0), (None, 0, 4.0, 4, 2, None, 0),
                 (None, 0, 4, 4, 2, None), (None, 0, 4, 4, 2, None, None)):
        with pytest.raises((TypeError, AttributeError)):
            n.bsp_mask_weights(*args)
    assert n.bsp_mask_weights(None, 0, 4, 4, 2, None, 0) == 1   # NULL: refused by the library
    # no tokens: accepted without looking at memory
    a, i = _Elsewhere(), _Elsewhere(torch.int32)
    assert n.bsp_linear_sized(a, 0, 0, 64, 64, 16, 32, i, i, i, a, 64, None, a, None, 0, 0) == 0
    assert n.bsp_linear_sized(a, 0, 0, 64, 64, 16, 32, i, i, i, a, -1, None, a, None, 0, 0) == 4
    assert n.bsp_linear_workspace_bytes(1, 4096, 1024, 4096, 16, 32, 1 << 17) == bsp.lib().bsp_linear_workspace_bytes(
        1, 4096, 1024, 4096, 16, 32, 1 << 17)
    assert n.empty(host, 3, 5).shape == (5,) and n.empty(host, 1, 2, 3).dtype == torch.bfloat16
    assert n.last(torch.tensor([3, 9, 7], dtype=torch.int32)) == 7
    with pytest.raises(RuntimeError):
        n.empty(host, 0, -1)


class _Index:
    def __index__(self):
        return 16


class _Named:
    def __init__(self, v):
        self._as_parameter_ = v


def test_native_functions_take_the_numbers_that_ctypes_takes():
    """A number in any form that the ctypes call of the same function accepts reaches the library (0: the call has no tokens; 3: 24
    rows are not whole row-blocks), and every other form is refused by both."""
    native, plain = bsp.bsp._native(), bsp.lib()
    a, i = _Elsewhere(), _Elsewhere(torch.int32)

    def both(M, R):
        return (native.bsp_linear_sized(a, 0, 0, M, 64, R, 32, i, i, i, a, 64, None, a, None, 0, 0),
                plain.bsp_linear_sized(4096, 0, 0, M, 64, R, 32, 4096, 4096, 4096, 4096, 64, None, 4096, None, 0, 0))
    for R in (16, np.int64(16), np.int32(16), np.uint8(16), torch.tensor(16), torch.tensor([16]), _Index(), _Named(16), _Named(_Index()),
              C.c_int32(16)):
        assert both(64, R) == (0, 0) and both(40, R) == (2, 2), R
    assert both(np.prod((4, 16)), 16) == (0, 0) and both(C.c_int64(64), 16) == (0, 0)
    for R in (16.0, np.float64(16), np.float32(16), torch.tensor(16.0), "16", None, C.c_float(16), _Named(16.0)):
        with pytest.raises(TypeError):
            native.bsp_linear_sized(a, 0, 0, 64, 64, R, 32, i, i, i, a, 64, None, a, None, 0, 0)
        with pytest.raises(C.ArgumentError):
            plain.bsp_linear_sized(4096, 0, 0, 64, 64, R, 32, 4096, 4096, 4096, 4096, 64, None, 4096, None, 0, 0)
    # the threshold, without a decision to make (NULL: refused by the library)
    for t in (0.5, 1, np.float32(0.5), np.int64(1), torch.tensor(0.5), _Index(), _Named(0.5), C.c_float(0.5)):
        assert native.bsp_prune_mask(None, 4, 4, t, -1, 0, None, None, None, 0, 0) == 1, t
        assert plain.bsp_prune_mask(None, 4, 4, t, -1, 0, None, None, None, 0, 0) == 1, t
    for t in ("0.5", None, C.c_double(0.5)):
        with pytest.raises(TypeError):
            native.bsp_prune_mask(None, 4, 4, t, -1, 0, None, None, None, 0, 0)
        with pytest.raises(C.ArgumentError):
            plain.bsp_prune_mask(None, 4, 4, t, -1, 0, None, None, None, 0, 0)


def test_a_number_that_stands_for_itself_is_refused():
    """An object that names itself as its _as_parameter_ ends as with ctypes, in a RecursionError and not on the stack."""
    a, i = _Elsewhere(), _Elsewhere(torch.int32)
    me = _Named(None)
    me._as_parameter_ = me
    for whole, real in ((me, 0.5), (64, me)):
        with pytest.raises(RecursionError):
            bsp.bsp._native().bsp_prune_mask(a, whole, 64, real, -1, 0, i, None, None, 0, 0)
    with pytest.raises(RecursionError):
        C.c_int64.from_param(me)


def test_results_are_allocated_without_the_interpreter_lock():
    """While a result is allocated other Python threads run: an allocation that takes long (here for its filling, on a GPU for hipMalloc
    or the cache's flush) does not hold them."""
    native, host = bsp.bsp._native(), torch.zeros(1)
    ticks, stop = [], threading.Event()

    def tick():
        while not stop.wait(0.001):
            ticks.append(time.perf_counter())
    deterministic = torch.are_deterministic_algorithms_enabled(), torch.is_deterministic_algorithms_warn_only_enabled()
    threads = torch.get_num_threads()
    thread = threading.Thread(target=tick)
    thread.start()
    try:
        torch.use_deterministic_algorithms(True)         # new memory is filled
        torch.set_num_threads(1)
        start = time.perf_counter()
        native.empty(host, 3, 1 << 30)
        end = time.perf_counter()
    finally:
        torch.use_deterministic_algorithms(deterministic[0], warn_only=deterministic[1])
        torch.set_num_threads(threads)
        stop.set()
        thread.join()
    if end - start < 0.05:
        pytest.skip("the allocation is too short to see another thread beside it")
    third = (end - start) / 3
    assert any(start + third < t < end - third for t in ticks)


def test_native_allocations_beside_an_object_that_is_no_plain_tensor():
    """Results lie on the device that such an object names, and its last element is read through its own methods."""
    class Vector:
        device = torch.device("cpu")

        def __getitem__(self, i):
            return torch.tensor([4, 6, 9])[i]

    class Sub(torch.Tensor):
        pass
    native = bsp.bsp._native()
    for like in (Vector(), torch.zeros(2).as_subclass(Sub), torch.nn.Parameter(torch.zeros(2)), torch.zeros(2)):
        a, b = native.empty(like, 4, 5), native.empty(like, 1, np.int64(2), 3)
        assert type(a) is torch.Tensor and a.shape == (5,) and a.dtype == torch.int32 and a.device.type == "cpu"
        assert type(b) is torch.Tensor and b.shape == (2, 3) and b.dtype == torch.bfloat16
    assert native.last(Vector()) == 9 and native.last(torch.tensor([3, 8], dtype=torch.int32).as_subclass(Sub)) == 8
    assert type(native.last(Vector())) is int
    with pytest.raises(AttributeError):
        native.empty(3.0, 4, 5)
    with pytest.raises(IndexError):
        native.last(torch.zeros(0, dtype=torch.int32))


def test_a_missing_native_module_is_built_alone(monkeypatch, tmp_path):
    """The library with the kernels does not need the module with the Python functions: without the module it is loaded as it is,
    and only the module is built, when it is needed."""
    from paper_2009_08065_amd import build
    built = []

    def refuse(*args, **kwargs):
        raise AssertionError("the kernels are compiled")
    monkeypatch.setattr(build, "HOST_LIB", str(tmp_path / "_bsp_host.so"))
    monkeypatch.setattr(build, "build", refuse)
    monkeypatch.setattr(build, "_compile", refuse)
    monkeypatch.setattr(build, "build_host", lambda: built.append("host"), raising=False)
    monkeypatch.setattr(bsp.bsp, "_LIB", None)
    monkeypatch.setattr(bsp.bsp, "_NATIVE", None)
    with pytest.warns(UserWarning, match="missing or older"):
        assert bsp.bsp.lib().bsp_version()
    assert built == []
    assert bsp.bsp._native().bsp_mask_weights(None, 0, 4, 4, 2, None, 0) == 1 and built == ["host"]
