"""Host-side checks of the C-ABI library (no GPU needed): it loads, exports
every function its headers declare, and validates configurations and
arguments before touching the device."""
import ctypes
import os
import re

import pytest

from paper_2505_18719_amd import inputs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def vla():
    from paper_2505_18719_amd import vla as binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2505_18719_amd import build
        build.build(verbose=False)
    binding.load_library()
    return binding


def _declared_functions():
    names = set()
    for f in os.listdir(os.path.join(ROOT, "include")):
        if f.endswith(".h"):
            txt = open(os.path.join(ROOT, "include", f)).read()
            names |= set(re.findall(r"^(?:int|void|const char\*|size_t)\s+(vla_\w+)\(", txt, re.M))
    return sorted(names)


@pytest.mark.parametrize("header", ["vla.h", "vla_learn.h", "vla_debug.h"])
@pytest.mark.parametrize("lang", ["c", "c++"])
def test_each_header_compiles_on_its_own(header, lang, tmp_path):
    """A C-ABI header includes what it uses: it compiles alone, as C99 and as
    C++, with warnings as errors (only the host compiler is needed)."""
    import shutil
    import subprocess
    cc = shutil.which("gcc" if lang == "c" else "g++")
    if cc is None:
        pytest.skip("no host compiler")
    src = tmp_path / ("h.c" if lang == "c" else "h.cpp")
    src.write_text(f'#include "{header}"\nint main(void) {{ return 0; }}\n')
    std = ["-std=c99", "-pedantic"] if lang == "c" else ["-std=c++17"]
    r = subprocess.run([cc, *std, "-Wall", "-Wextra", "-Werror", "-fsyntax-only", "-I", os.path.join(ROOT, "include"),
                        str(src)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr


def test_headers_declare_the_rollout_entry_points():
    names = _declared_functions()
    for n in ("vla_prefill", "vla_decode_actions", "vla_token_logprobs", "vla_create", "vla_workspace_size",
              "vla_destroy", "vla_last_error"):
        assert n in names


def test_library_exports_every_declared_symbol(vla):
    lib = vla.load_library()
    missing = [n for n in _declared_functions() if not hasattr(lib, n)]
    assert not missing, missing


def test_workspace_size_and_config_validation(vla):
    lib = vla.load_library()
    n = ctypes.c_size_t()
    c = vla.make_config(inputs.L7B_B64, max_batch=64)
    assert lib.vla_workspace_size(ctypes.byref(c), ctypes.byref(n)) == 0
    # repacked weights (~13.2 GB incl. embedding) + KV pool for 64 x 320 tokens (~10.7 GB) + activations
    assert 20e9 < n.value < 40e9
    bad = [dict(head_dim_override=96), dict(max_seq=400), dict(action_bins=300), dict(max_batch=0),
           dict(n_actions=0), dict(page_size=8)]
    for b in bad:
        c = vla.make_config(inputs.TINY)
        for k, v in b.items():
            setattr(c, "head_dim" if k == "head_dim_override" else k, v)
        rc = lib.vla_workspace_size(ctypes.byref(c), ctypes.byref(n))
        assert rc in (-1, -7), (b, rc)
        assert lib.vla_last_error().decode()
    assert lib.vla_workspace_size(None, ctypes.byref(n)) == -1


def test_create_rejects_null_arguments_before_device_work(vla):
    lib = vla.load_library()
    c = vla.make_config(inputs.TINY)
    h = ctypes.c_void_p()
    assert lib.vla_create(ctypes.byref(c), None, None, 0, None, ctypes.byref(h)) == -1
    assert "NULL" in lib.vla_last_error().decode()
    assert lib.vla_prefill(None, 1, None, None, None, None, None) == -1
    assert lib.vla_decode_actions(None, 1, None, 1.0, None, None, None, None, None) == -1
    lib.vla_destroy(None)


def test_lora_merge_validates_arguments_before_the_device(vla):
    """Null handle, unknown projection, bad rank or scale are rejected by the
    host code (no model or device memory is touched)."""
    lib = vla.load_library()
    p = ctypes.c_void_p(16)  # never dereferenced: validation fails first
    assert lib.vla_lora_merge(None, 0, 0, p, p, p, 8, 1.0, None) == -1
    assert b"model is NULL" in lib.vla_last_error()
    arr = (ctypes.c_void_p * 7)(*([p] * 7))
    assert lib.vla_lora_merge_layer(None, 0, arr, arr, arr, 8, 1.0, None) == -1
    assert b"model is NULL" in lib.vla_last_error()


def test_learning_entry_points_validate_on_the_host(vla):
    """vla_learn.h: bad sizes, parameters and null buffers are rejected, and
    empty windows are no-ops, all before any device work."""
    lib = vla.load_library()
    p = ctypes.c_void_p(16)  # never dereferenced: validation fails first
    assert lib.vla_gae(4, 8, p, p, p, 1.5, 0.9, p, p, None) == -1
    assert b"gamma" in lib.vla_last_error()
    assert lib.vla_gae(4, 8, p, p, p, 0.99, float("nan"), p, p, None) == -1
    assert lib.vla_gae(-1, 8, p, p, p, 0.99, 0.9, p, p, None) == -1
    assert lib.vla_gae(0, 8, None, None, None, 0.99, 0.9, None, None, None) == 0
    assert lib.vla_gae(4, 0, None, None, None, 0.99, 0.9, None, None, None) == 0
    assert lib.vla_gae(4, 8, p, None, p, 0.99, 0.9, p, None, None) == -1
    assert lib.vla_ppo_clip(0, 7, p, p, p, 0.2, p, p, None) == -1
    assert lib.vla_ppo_clip(4, 17, p, p, p, 0.2, p, p, None) == -1
    assert lib.vla_ppo_clip(4, 7, p, p, p, -0.1, p, p, None) == -1
    assert lib.vla_ppo_clip(4, 7, p, p, p, float("inf"), p, p, None) == -1
    assert lib.vla_ppo_clip(4, 7, p, p, None, 0.2, p, p, None) == -1
    assert lib.vla_logprob_backward(4, 257, 0, p, p, 1.0, p, p, None) == -7
    assert lib.vla_logprob_backward(4, 256, 0, p, p, 0.0, p, p, None) == -1
    assert lib.vla_logprob_backward(0, 256, 0, None, None, 1.5, None, None, None) == 0
    assert lib.vla_logprob_backward(4, 256, 0, p, None, 1.5, p, p, None) == -1


class _SkinnyPlan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("tiles", "chunks", "G", "dp_tiles", "slots")]


@pytest.mark.parametrize("N,K,workgroups", [(30000 * 64, 512, 40000), (32000 * 64, 512, 1 << 30), (4096, 11008, 256),
                                            (12288, 4096, 256), (16000 * 64, 1024, 20000), (64, 256, 100000)])
def test_decode_gemm_plan_stays_in_32_bit_units(vla, N, K, workgroups):
    """The decode GEMM's kernels form (workgroup + 1) * units and unit * workgroups in 32 bits: no plan goes past them,
    whatever number of workgroups is asked for, and each tile's closed-form slot count is the one of exact arithmetic."""
    plan = vla.load_library()["_ZN3vla11skinny_planEiiii"]
    plan.restype, plan.argtypes = _SkinnyPlan, [ctypes.c_int] * 4
    p = plan(N, K, workgroups, 16)
    assert (p.tiles, p.chunks) == (N // 64, K // 256) and 1 <= p.G <= workgroups
    assert p.dp_tiles == p.tiles // p.G * p.G
    U = (p.tiles - p.dp_tiles) * p.chunks
    assert U == 0 or U >= p.G
    assert (U + 1) * p.G + U < 2 ** 31
    slots = 1
    for t in range(p.tiles - p.dp_tiles):
        first, last = (((u + 1) * p.G + U - 1) // U - 1 for u in (t * p.chunks, (t + 1) * p.chunks - 1))
        slots = max(slots, last - first + 1)
    assert p.slots == slots <= 16


class _GemmPlan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("first", "rest", "rows", "cols")]


def test_prefill_gemm_plan_keeps_full_rounds_on_the_large_tile(vla):
    """From one round of 256 x 256 tiles per CU on, a smaller tile shape takes a whole product only where the second round
    is nearly empty, and a cut's rest is less than half a round (gate/up of d = 256 and 200 environments ran 64 x 64 tiles
    for 5 rounds: 137 us, 82 on the large tile); below one round, few rows run smaller tiles."""
    plan = vla.load_library()["_ZN3vla9gemm_planEiiiiNS_12GemmEpilogueE"]
    plan.restype, plan.argtypes = _GemmPlan, [ctypes.c_int] * 5
    store, residual, swiglu, qkv, keep = range(5)
    cuts = whole = 0
    for d, f in ((256, 688), (512, 1376), (1024, 2752), (1280, 3400), (2048, 5504), (4096, 11008)):
        fp = 32 * -(-f // 32)
        for M in (277, 1108, 4432, 6656, 8864, 17728, 22160, 35456, 55400, 141824):
            for N, K, epi in ((3 * d, d, qkv), (d, d, residual), (2 * fp, d, swiglu), (2 * fp, d, keep), (d, fp, residual),
                              (fp, d, store)):
                p = plan(M, N, K, 256, epi)
                tiles = -(-M // 256) * -(-N // 256)
                assert 0 <= p.first <= 8 and 0 <= p.rest <= 8
                if p.rows or p.cols:
                    cuts += 1
                    assert p.first == 0 and p.rest >= 1 and not (p.rows and p.cols)
                    assert 0 <= p.rows < M and 0 <= p.cols < N and p.rows % 256 == 0 and p.cols % 256 == 0
                    assert tiles >= 256 and tiles % 256 < 128, (M, N, K, epi)
                    assert K >= 512 or (epi not in (swiglu, keep) and tiles < 3 * 256)
                elif p.first:
                    whole += 1
                    assert tiles <= 256 * (1.2 if epi == qkv else 1.25), (M, N, K, epi)
    assert cuts >= 20 and whole >= 50
    assert plan(55200, 1408, 256, 256, swiglu).first == 0 and plan(277, 4096, 4096, 256, residual).first > 0


def test_extract_actions_validates_on_the_host(vla):
    lib = vla.load_library()
    p = ctypes.c_void_p(16)  # never dereferenced: validation fails first
    assert lib.vla_extract_actions(4, 0, p, 0, 256, p, p, p, None) == -1
    assert lib.vla_extract_actions(4, 7, p, 0, 300, p, p, p, None) == -7
    assert lib.vla_extract_actions(4, 7, p, 0, 256, None, p, p, None) == -1
    assert lib.vla_extract_actions(0, 7, None, 0, 256, None, None, None, None) == 0


def test_lora_gradient_entry_validates_on_the_host(vla):
    """vla_ppo_lora_grads rejects a NULL model, bad batch, rank, parameters and a
    missing workspace before any device work."""
    lib = vla.load_library()
    p = ctypes.c_void_p(16)  # never dereferenced: validation fails first
    lora = vla._Lora(8, 0.5, None, None, None, None)
    assert lib.vla_ppo_lora_grads(None, 1, p, p, p, p, p, p, 0.2, 1.5, ctypes.byref(lora), p, 1, p, None, None) == -1
    assert b"model is NULL" in lib.vla_last_error()
    n = ctypes.c_size_t()
    c = vla.make_config(inputs.TINY)
    assert lib.vla_train_workspace_size(ctypes.byref(c), 0, ctypes.byref(n)) == 0 and n.value > 0
    n_keep = ctypes.c_size_t()
    assert lib.vla_train_workspace_size(ctypes.byref(c), 1, ctypes.byref(n_keep)) == 0 and n_keep.value > n.value
    assert lib.vla_train_workspace_size(ctypes.byref(c), 2, ctypes.byref(n)) == -1
    assert lib.vla_train_workspace_size(None, 0, ctypes.byref(n)) == -1
