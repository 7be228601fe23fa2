"""Host-only checks of the boundary: the C-ABI library loads without a GPU, exports every
symbol the header declares, and its pure-host entry points behave as documented."""
import ctypes
import os
import re

import pytest
import torch

from paper_2104_11125_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_symbols():
    text = open(os.path.join(ROOT, "include", "scalecom.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(scalecom_[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    L = binding.lib()
    names = _declared_symbols()
    assert {"scalecom_init", "scalecom_step", "scalecom_step_layers", "scalecom_workspace_bytes",
            "scalecom_strerror", "scalecom_last_error", "scalecom_destroy"} <= set(names)
    for name in names:
        assert getattr(L, name) is not None


def test_header_is_plain_c(tmp_path):
    """The boundary's header compiles as C99 on its own (no C++ or torch types in the signatures)."""
    import shutil
    import subprocess
    gcc = shutil.which("gcc")
    assert gcc, "gcc is part of the image"
    src = tmp_path / "abi.c"
    src.write_text('#include "scalecom.h"\nint main(void) { return (int)scalecom_workspace_bytes(0, 1, 1, 0); }\n')
    res = subprocess.run([gcc, "-std=c99", "-Wall", "-Wextra", "-pedantic", "-Werror", "-I", os.path.join(ROOT, "include"),
                          "-c", str(src), "-o", str(tmp_path / "abi.o")], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr


def test_hamming_scratch_bytes_is_host_arithmetic():
    L = binding.lib()
    small = L.scalecom_hamming_scratch_bytes(1_000_000, 1)
    large = L.scalecom_hamming_scratch_bytes(100_000_000, 200)
    assert 4 * 1_000_000 < small < 5 * 1_000_000          # the summed vector + one bit per position + predictions
    assert small < large < 5 * 100_000_000
    assert L.scalecom_hamming_scratch_bytes(-1, 1) == 0 and L.scalecom_hamming_scratch_bytes(10, 0) == 0
    assert L.scalecom_hamming_distance(None, None, None, 1, 1, None, None, 0.1, 0, None, 0, None) == binding.SCALECOM_EINVAL
    assert L.scalecom_cosine_distance(None, None, None, 0, None) == binding.SCALECOM_EINVAL
    assert L.scalecom_step_layers_chunked(None, None, None, 1, 1, None, None, 0.5, 0.1, 0, None, None) == binding.SCALECOM_EINVAL


def test_workspace_bytes_is_host_arithmetic():
    small = binding.scalecom_workspace_bytes(1_048_576, 1, 4, 10_485)
    large = binding.scalecom_workspace_bytes(1_000_000_000, 1, 8, 2_500_000)
    layered = binding.scalecom_workspace_bytes(1_048_576, 200, 4, 10_485)
    more_k = binding.scalecom_workspace_bytes(1_048_576, 1, 4, 1_048_576)
    assert 0 < small < large and small < layered and small < more_k
    assert large < 1_000_000_000                      # below one byte per element
    assert binding.scalecom_workspace_bytes(-1, 1, 1, 0) == 0
    assert binding.scalecom_workspace_bytes(2 ** 31, 1, 1, 0) == 0     # positions are int32
    assert binding.scalecom_workspace_bytes(10, 0, 1, 0) == 0
    assert binding.scalecom_workspace_bytes(10, 1, 65, 0) == 0
    assert binding.scalecom_workspace_bytes(10, 1, 1, 11) == 0


def test_workspace_size_as_the_header_states_it():
    """No more than the header's formula: the parts of a short layout are counted once, and a part that is partly empty only with
    as many positions as a layout of that length can give it."""
    for numel, tensors, learners in [(1_048_576, 1, 4), (25_557_032, 1, 8), (60_000, 60, 4), (2_400_000, 60, 4), (8_000_000, 1_000, 4),
                                     (120_000_000, 200, 8), (1_000_000_000, 1, 8), (0, 1, 1)]:
        k = numel // 100
        short = 8 * min(numel, (2 if tensors == 1 else 8) << 20)
        got = binding.scalecom_workspace_bytes(numel, tensors, learners, k)
        assert 0 < got <= 0.8 * numel + short + (4 * learners + 16) * k + 170 * 1024 * tensors + 600 * 1024, (numel, tensors)


def test_argument_checks_that_need_no_device():
    L = binding.lib()
    out = ctypes.c_void_p()
    assert L.scalecom_init(None, 0, None, None, 0, 1, 10, 10, 1, 0) == binding.SCALECOM_EINVAL
    assert L.scalecom_init(ctypes.byref(out), 0, None, None, 0, 1, 10, 10, 1, 0) == binding.SCALECOM_EINVAL   # no workspace
    assert L.scalecom_init(ctypes.byref(out), 0, None, ctypes.c_void_p(256), 1 << 30, 65, 10, 10, 1, 0) == binding.SCALECOM_EINVAL
    assert L.scalecom_init(ctypes.byref(out), 0, None, ctypes.c_void_p(256), 1 << 30, 1, 10, 11, 1, 0) == binding.SCALECOM_EINVAL
    assert L.scalecom_init(ctypes.byref(out), 0, None, ctypes.c_void_p(256), 16, 1, 10, 10, 1, 0) == binding.SCALECOM_ENOMEM
    assert L.scalecom_init(ctypes.byref(out), 0, None, ctypes.c_void_p(256), 1 << 30, 1, 10, 10, 1, 7) == binding.SCALECOM_EINVAL
    assert out.value is None
    assert L.scalecom_step(None, None, None, 1, 1, 1, 0.5, 0.1, 0, None, None) == binding.SCALECOM_EINVAL
    assert L.scalecom_strerror(0) == b"ok" and b"invalid" in L.scalecom_strerror(1)
    assert L.scalecom_last_error(None) == b""
    L.scalecom_destroy(None)


def test_static_entry_point_checks_that_need_no_device():
    """scalecom_step_static refuses what its static workspace cannot hold, and malformed arguments,
    before it touches a device; the reason is the calling thread's scalecom_last_error(NULL)."""
    L = binding.lib()
    fake = (ctypes.c_void_p * 8)(*([256] * 8))               # never dereferenced: every call below fails first
    vp = lambda x: ctypes.c_void_p(x)

    def call(device=0, n=2, numel=1000, k=10, beta=0.5, lr=0.1, step=0, dtype=0, mem=fake, grad=fake, idx=vp(256), red=vp(256)):
        return L.scalecom_step_static(device, None, mem, grad, n, numel, k, beta, lr, step, dtype, idx, red)

    cases = [(dict(device=-1), b"device"), (dict(device=64), b"device"), (dict(dtype=7), b"grad_dtype"),
             (dict(numel=binding.SCALECOM_STATIC_NUMEL_MAX + 1), b"SCALECOM_STATIC_NUMEL_MAX"), (dict(numel=-1), b"numel"),
             (dict(n=binding.SCALECOM_STATIC_LEARNERS_MAX + 1), b"SCALECOM_STATIC_LEARNERS_MAX"), (dict(n=0), b"n_learners"),
             (dict(k=1001), b"k must"), (dict(k=-1), b"k must"),
             (dict(numel=binding.SCALECOM_STATIC_NUMEL_MAX, k=binding.SCALECOM_STATIC_K_MAX + 1), b"SCALECOM_STATIC_K_MAX"),
             (dict(beta=0.0), b"beta"), (dict(beta=1.5), b"beta"), (dict(beta=float("nan")), b"beta"),
             (dict(lr=float("inf")), b"lr"), (dict(step=-1), b"step"), (dict(mem=None), b"null"), (dict(grad=None), b"null"),
             (dict(idx=None), b"null output"), (dict(red=None), b"null output")]
    for kwargs, word in cases:
        assert call(**kwargs) == binding.SCALECOM_EINVAL, kwargs
        assert word in L.scalecom_last_error(None), (kwargs, L.scalecom_last_error(None))
    assert call(numel=0, k=0) == binding.SCALECOM_OK          # nothing to do, nothing touched
    assert L.scalecom_last_error(None) == b""
    assert L.scalecom_selection_stats(None, None, 0) == binding.SCALECOM_EINVAL


def test_static_binding_refuses_learners_without_a_gradient(monkeypatch):
    """Fewer gradients than memories: refused before anything is handed to the library, whose pointer tables
    would otherwise end before the learner count that goes with them.  (Further gradients are ignored.)"""
    handed = []

    class Lib:
        def scalecom_step_static(self, index, stream, mem, grad, n, *rest):
            handed.append((len(mem), len(grad), n))
            return binding.SCALECOM_OK

    class Stream:
        cuda_stream = 0

    monkeypatch.setattr(binding, "lib", lambda: Lib())
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    bufs = [torch.zeros(8) for _ in range(3)]
    idx, red = torch.zeros(2, dtype=torch.int32), torch.zeros(2)
    with pytest.raises(ValueError):
        binding.scalecom_step_static(bufs, bufs[:1], 2, 0.5, 0.1, 0, idx, red, stream=Stream())
    assert handed == []
    binding.scalecom_step_static(bufs[:2], bufs, 2, 0.5, 0.1, 0, idx, red, stream=Stream())
    assert handed == [(2, 2, 2)]


def test_workloads_match_the_benchmark_table():
    from paper_2104_11125_amd import workloads
    cfg = {w.name: w for w in workloads.configs()}
    assert cfg["tiny"].k == 10_485 and cfg["resnet50_sized"].k == 228_187
    assert cfg["transformer_base_sized"].k == 275_000 and cfg["large_bf16"].k == 2_500_000
    pl = cfg["per_layer"]
    assert pl.n_tensors == 200 and len(pl.offsets) == 201 and all(64 <= b - a <= 4_194_304 for a, b in zip(pl.offsets, pl.offsets[1:]))
    assert all(k == -(-(b - a) // 100) for k, a, b in zip(pl.ks, pl.offsets, pl.offsets[1:]))


def test_layer_ks_follows_the_rate_guidance():
    import oracle
    ratios = [3000.0, 196.0, 150.0, 128.0, 64.0, 0.5]
    sizes = [1_000_000, 25, 4097, 50, 400, 0]
    ks, rates = binding.scalecom_layer_ks(ratios, sizes)
    assert rates == [25, 25, 50, 50, 400, 400] == [oracle.layer_rate(r) for r in ratios]
    assert ks == [40_000, 1, 82, 1, 1, 0]
    # layers kept out of compression send everything (App. E: first convolution; warm-up epochs)
    ks, rates = binding.scalecom_layer_ks(ratios, sizes, [True, False, False, True, False, True])
    assert rates == [1, 25, 50, 1, 400, 1] and ks == [1_000_000, 1, 82, 50, 1, 0]
    L = binding.lib()
    assert L.scalecom_layer_ks(1, None, None, None, None, None) == binding.SCALECOM_EINVAL
    bad = (ctypes.c_double * 1)(0.0); one = (ctypes.c_int64 * 1)(5); out = (ctypes.c_int64 * 1)()
    assert L.scalecom_layer_ks(1, bad, one, None, out, None) == binding.SCALECOM_EINVAL
    assert L.scalecom_apply_update(None, None, 0, None, None, 0, 1.0) == binding.SCALECOM_EINVAL


def test_bench_refuses_more_than_one_gpu():
    """bench.py runs on one GPU; asked for more it says so and exits non-zero before touching a device."""
    import subprocess
    import sys
    res = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True,
                         timeout=120)
    assert res.returncode != 0
    assert "ONE GPU" in res.stderr
    assert res.stdout.strip() == ""
