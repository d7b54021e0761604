"""Waits in the assembly of the kernels that copy into LDS behind the compiler's
back (compiled for gfx950, nothing is run).  A wave that crosses a workgroup
barrier with LDS reads in flight lets the other waves' next copies overwrite what
it has not read yet, so the last LDS instruction before every barrier has to be
followed by a wait for all of them (lgkmcnt(0))."""
import importlib.util
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _assembly(source, tmp_path):
    """{function: its lines} of one device source (or source text)."""
    spec = importlib.util.spec_from_file_location("rqc_build", os.path.join(ROOT, "paper_2110_14502_amd", "build.py"))
    b = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(b)
    try:
        hipcc = b._hipcc()
    except RuntimeError:
        pytest.skip("hipcc not available")
    out = str(tmp_path / "k.s")
    r = subprocess.run([hipcc] + b.COMMON + b.DEVICE + ["--cuda-device-only", "-S", source, "-o", out],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    funcs, name = {}, None
    for line in open(out):
        m = re.match(r"^(_Z\w+):", line)
        if m:
            name = m.group(1)
        if name:
            funcs.setdefault(name, []).append(line.split(";")[0].strip())
    return funcs


def _source(name):
    return os.path.join(ROOT, "paper_2110_14502_amd", "csrc", name)


@pytest.mark.parametrize("source,kernel,n_kernels", [("k_gemm16.hip", "k_frag_gemm", 2), ("k_split32.hip", "k_frag_gemm", 1),
                                                     ("k_mfma32.hip", "k_mfma32_copy", 4)])
def test_lds_reads_end_before_barriers(source, kernel, n_kernels, tmp_path):
    found = 0
    for name, lines in _assembly(_source(source), tmp_path).items():
        if kernel not in name or not any("s_barrier" in x for x in lines):
            continue
        found += 1
        for at, line in enumerate(lines):
            if line != "s_barrier":
                continue
            for before in reversed(lines[:at]):
                if before.startswith("s_waitcnt") and "lgkmcnt(0)" in before:
                    break
                # (a lane exchange goes through the LDS unit but not its memory)
                assert not before.startswith("ds_") or before.startswith("ds_bpermute"), (name, at, before)
    assert found == n_kernels


def test_copies_into_lds_name_m0(tmp_path):
    """lds_copy16 overwrites M0: a value that the compiler keeps there (its own
    copies into LDS address by M0) has to be set again behind it."""
    src = tmp_path / "probe.hip"
    src.write_text("""
#include "kernels_dev.h"
using namespace rqc;
__global__ void probe(const float4* p, float4* out) {
  __shared__ float4 own[64], other[64];
  typedef __attribute__((address_space(1))) const void global_t;
  typedef __attribute__((address_space(3))) void lds_t;
  __builtin_amdgcn_global_load_lds((global_t*)(p + threadIdx.x), (lds_t*)own, 4, 0, 0);
  lds_copy16(p + 64 + threadIdx.x, lds_address(other));
  __builtin_amdgcn_global_load_lds((global_t*)(p + 128 + threadIdx.x), (lds_t*)own, 4, 64, 0);
  __syncthreads();
  out[threadIdx.x] = own[threadIdx.x];
}
""")
    (lines,) = [v for k, v in _assembly(str(src), tmp_path).items() if "probe" in k]
    state = [re.split(r"[ ,]", x)[0] if "global_load_lds" in x else "m0" for x in lines
             if "global_load_lds" in x or re.match(r"s_mov_b32 m0,", x)]
    copies = [i for i, x in enumerate(state) if x != "m0"]
    assert len(copies) == 3 and all(state[i - 1] == "m0" for i in copies), state
