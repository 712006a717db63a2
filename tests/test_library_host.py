"""Host-side checks of libdartqr.so that need no GPU: it loads, exports every entry point that
include/dartqr.h declares, and its argument checks refuse bad calls before anything is launched."""

import ctypes
import os
import re
import subprocess

import pytest

from paper_2511_04063_amd import binding as B
from paper_2511_04063_amd.build import HIPCC_FLAGS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(B.LIB_PATH):
        from paper_2511_04063_amd.build import build_library
        build_library(verbose=False)
    return B.load_library()


def declared_entry_points():
    text = open(os.path.join(ROOT, "include", "dartqr.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(dq_[a-z0-9_]+)\s*\(", text)))


def test_header_symbols_are_exported_and_bound(lib):
    names = declared_entry_points()
    assert {"dq_qr_orth", "dq_rotate_loss_grad", "dq_calib_step"} <= set(names)
    for name in names:
        assert hasattr(lib, name), f"{name} declared in dartqr.h but not exported"
        assert name in B.SIGNATURES, f"{name} has no binding"
    assert sorted(B.SIGNATURES) == names


def test_status_strings(lib):
    seen = {B.status_string(s) for s in range(0, 8)}
    assert len(seen) == 8 and "ok" in seen
    assert B.status_string(99) == "unknown status"


def test_workspace_bytes_rules(lib):
    small = B.workspace_bytes(1, 256, 2048, B.DQ_F32)
    big = B.workspace_bytes(1, 4096, 8192, B.DQ_BF16)
    assert 0 < small < big
    assert small % 256 == 0
    # batches run one after another: the workspace does not grow with b ...
    assert B.workspace_bytes(64, 256, 16384, B.DQ_BF16) == B.workspace_bytes(1, 256, 16384, B.DQ_BF16)
    # ... except for 128 x 128 rotations, whose problems all run in the same launches: 7 matrices and
    # ceil(T / 2048) partial gradients per problem
    w1, w64 = B.workspace_bytes(1, 128, 16384, B.DQ_BF16), B.workspace_bytes(64, 128, 16384, B.DQ_BF16)
    assert w1 < w64 and w64 - w1 == 63 * (7 + 8) * 128 * 128 * 4 + (64 * 8 * 8 - 256)
    # the 70B-shaped problem fits comfortably in one GPU's HBM
    assert B.workspace_bytes(1, 8192, 16384, B.DQ_BF16) < 8 * 2 ** 30
    out = ctypes.c_size_t(0)
    assert lib.dq_workspace_bytes(1, 0, 16, B.DQ_F32, ctypes.byref(out)) == B.DQ_ERR_SHAPE
    assert lib.dq_workspace_bytes(1, B.DQ_MAX_N + 1, 16, B.DQ_F32, ctypes.byref(out)) == B.DQ_ERR_UNSUPPORTED
    assert lib.dq_workspace_bytes(1, 16, 0, B.DQ_F32, ctypes.byref(out)) == B.DQ_ERR_SHAPE
    assert lib.dq_workspace_bytes(-1, 16, 16, B.DQ_F32, ctypes.byref(out)) == B.DQ_ERR_SHAPE
    assert lib.dq_workspace_bytes(1, 16, 16, 7, ctypes.byref(out)) == B.DQ_ERR_DTYPE
    assert lib.dq_workspace_bytes(1, 16, 16, B.DQ_F32, None) == B.DQ_ERR_NULL


def test_null_context_is_refused_everywhere(lib):
    z = ctypes.c_void_p(0)
    assert lib.dq_destroy(z) == B.DQ_ERR_NULL
    assert lib.dq_set_workspace(z, z, 0) == B.DQ_ERR_NULL
    assert lib.dq_device_flags(z, None) == B.DQ_ERR_NULL
    assert lib.dq_qr_orth(z, 1, 8, z, 8, z, 8, z, 8) == B.DQ_ERR_NULL
    assert lib.dq_rotate_loss_grad(z, 1, 8, 8, z, 0, 8, z, 8, 0, z, z, 8, z, 8, z, 8) == B.DQ_ERR_NULL
    assert lib.dq_calib_step(z, 1, 8, 8, z, 0, 8, z, 8, 0.1, 0, z, z, 8) == B.DQ_ERR_NULL
    assert lib.dq_qr_backward(z, 1, 8, z, 8, z, 8, z, 8, z, 8) == B.DQ_ERR_NULL
    assert lib.dq_whip_loss_grad(z, 1, 8, 8, z, 8, 0, z, z, 0, 8) == B.DQ_ERR_NULL
    assert lib.dq_objective_loss_grad(z, 1, 4, 1, 8, 8, z, 8, 0, z, z, 0, 8) == B.DQ_ERR_NULL
    assert lib.dq_set_objective(z, 1, 4) == B.DQ_ERR_NULL
    assert lib.dq_calib_run_host_batches(z, 8, 8, z, 1, 0, 8, z, z, 8, 0.1, 0, 1, z) == B.DQ_ERR_NULL
    assert lib.dq_sgd_update(z, 1, 8, z, 8, z, 8, 0.1) == B.DQ_ERR_NULL
    assert lib.dq_gemm_f32(z, 8, 8, 8, 1.0, z, 8, 0, z, 8, 0, 0.0, z, 8) == B.DQ_ERR_NULL
    assert lib.dq_gemm_bf16(z, 8, 8, 8, z, 8, 0, z, 8, 0, z, 8) == B.DQ_ERR_NULL
    assert lib.dq_profile_enable(z, 1) == B.DQ_ERR_NULL
    assert lib.dq_profile_read(z, 0, None, None, None, None) == B.DQ_ERR_NULL
    assert lib.dq_create(None, z) == B.DQ_ERR_NULL


def test_missing_library_fails_loudly(tmp_path):
    with pytest.raises(RuntimeError, match="no CPU fallback"):
        B.load_library(str(tmp_path / "libdartqr.so"))


def test_workspace_of_small_batches():
    """A batch of small rotations asks for matrices of its own order and for no more than a group of problems."""
    one = B.workspace_bytes(1, 16, 512, B.DQ_BF16)
    many = B.workspace_bytes(4096, 16, 512, B.DQ_BF16)
    # 1024 problems: four 16 x 16 matrices and up to 16 partial gradients of 32 x 32 each
    assert many - one <= 1024 * (4 * 1024 + 16 * (4096 + 8))
    assert B.workspace_bytes(100000, 16, 512, B.DQ_BF16) == many
    assert B.workspace_bytes(64, 128, 16384, B.DQ_BF16) - B.workspace_bytes(1, 128, 16384, B.DQ_BF16) <= 63 * 15 * 65536 + 63 * 64


def test_stores_have_arrived_before_a_signal(tmp_path):
    """Workgroups hand data to each other by a word that one thread sets behind a barrier.  Every wavefront has to wait for its own stores
    in front of that barrier: the thread's release waits for its own wavefront's only."""
    csrc = os.path.join(ROOT, "paper_2511_04063_amd", "csrc")
    arrivals = 0
    for name in ("qr_gram.hip", "qr_cholpanel.hip"):
        lines = open(os.path.join(csrc, name)).read().splitlines()
        for i, line in enumerate(lines):
            if re.search(r"fetch_add\(.*__ATOMIC_RELEASE|handover_signal\((ready|ps\.)", line):
                arrivals += 1
                assert any("store_barrier();" in before for before in lines[i - 2:i]), f"{name}:{i + 1}"
    assert arrivals == 8
    src, out = tmp_path / "k.hip", tmp_path / "k.s"
    src.write_text('#include "dq_internal.h"\n'
                   "__global__ void k(float* a, unsigned long long* word) {\n"
                   "    a[threadIdx.x] = 1.f;\n"
                   "    dq::store_barrier();\n"
                   "    if (threadIdx.x == 0) dq::handover_signal(word, 1ull);\n"
                   "}\n")
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *HIPCC_FLAGS, "--cuda-device-only", "-S", "-w", "-I", csrc,
                    "-I", os.path.join(ROOT, "include"), str(src), "-o", str(out)], check=True, capture_output=True)
    code = [w for w in re.findall(r"global_store_dword\b|s_waitcnt vmcnt\(0\)|s_barrier|global_store_dwordx2|buffer_wbl2", out.read_text())]
    assert code[:5] == ["global_store_dword", "s_waitcnt vmcnt(0)", "s_barrier", "buffer_wbl2", "s_waitcnt vmcnt(0)"]
