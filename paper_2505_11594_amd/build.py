"""Build the gfx950 HIP library ``libsage_mi355x.so`` in-tree with hipcc, the
separate measurement library ``libsage_rates.so`` (instruction issue-rate
microbenchmarks used by ``bench.py --mode rates``) and the hardware-probe
library ``libsage_probes.so`` (the conversion, exp2 and MFMA-layout semantics
the kernels rely on, checked by the tests).

Every HIP source is compiled for ``--offload-arch=gfx950`` only.  Packed FP32
instructions are disabled (``-packed-fp32-ops``) and floating-point
contraction is off: the kernels spell out every fused multiply-add they use,
because the quantization decisions must round exactly like the definition.
"""
from __future__ import annotations

import concurrent.futures
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsage_mi355x.so")
SOURCES = ["sage_abi.hip", "quant.hip", "attn_fp4.hip", "attn_bf16.hip", "attn_nv16.hip", "quant_int8.hip",
           "attn_int8.hip", "attn_int8_bwd.hip"]
RATES_LIB = os.path.join(HERE, "libsage_rates.so")
RATES_SOURCES = ["issue_rates.hip"]
PROBES_LIB = os.path.join(HERE, "libsage_probes.so")
PROBES_SOURCES = ["probes.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-result",
    "-I" + os.path.join(ROOT, "include"),
]


# MFMA results in VGPRs: where LDS allows one workgroup per CU only (two KV groups
# of 256-key tiles), the compiler counts on 512 registers, puts the scores into
# AGPRs and moves each one back before its use (32 -> 28 us on 4 heads x 4096, D =
# 128).  The other FP4 kernels use no AGPR either way.
SOURCE_FLAGS = {"attn_fp4.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"]}


def _run(cmd, verbose: bool) -> None:
    r = subprocess.run(cmd, capture_output=True, text=True)
    # the host pass does not know the device-only feature name; that warning is harmless
    msgs = [l for l in (r.stdout + r.stderr).splitlines() if "not a recognized feature" not in l]
    if r.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + "\n".join(msgs))
    if verbose and msgs:
        print("\n".join(msgs), file=sys.stderr)


def _compile(lib: str, sources, verbose: bool) -> str:
    tmp = lib + ".tmp%d" % os.getpid()
    with tempfile.TemporaryDirectory() as d, concurrent.futures.ThreadPoolExecutor(4) as pool:
        objs = [os.path.join(d, s + ".o") for s in sources]
        list(pool.map(lambda so: _run([HIPCC] + FLAGS + SOURCE_FLAGS.get(so[0], []) +
                                      ["-c", "-o", so[1], os.path.join(CSRC, so[0])], verbose), zip(sources, objs)))
        _run([HIPCC, "--offload-arch=gfx950", "-fPIC", "-shared", "-o", tmp] + objs, verbose)
    os.replace(tmp, lib)
    return lib


def build(verbose: bool = False) -> str:
    _compile(RATES_LIB, RATES_SOURCES, verbose)
    _compile(PROBES_LIB, PROBES_SOURCES, verbose)
    return _compile(LIB, SOURCES, verbose)


if __name__ == "__main__":
    print(build(verbose=True))
