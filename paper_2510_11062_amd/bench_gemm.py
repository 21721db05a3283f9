"""The tile loop of the bf16 head kernels as plain GEMMs beside the vendor GEMM (hipBLASLt through torch.mm) on the
shapes the library launches.

    python -m paper_2510_11062_amd.bench_gemm

One JSON line per case: variant, shape, TFLOP/s, shader clock.  Shapes (bf16, fp32 accumulate):
  logits         vocabulary x tokens of one launch x H          151808 x 16384 x 2048   (short k)
  dHidden        H x tokens x vocabulary                         2048 x 16384 x 151936   (long k)
  dW             H x vocabulary x tokens of a super-chunk, both operands k-major  2048 x 151808 x 32768
  a square case  8192^3
The suffix of a variant is the wavefront grid: 8 = 4 x 2, t = 2 x 4, 4 = 2 x 2; the library uses ntt for the logits, nt4
for dHidden and km8 for dW; mx4 is dHidden on untransposed weights.  The probe (csrc/gemm_probe.hip, built by
build.py) runs the library's own loop without any epilogue; torch.mm is timed with the output written.  A measurement
aid: nothing in the library calls this.
"""
from __future__ import annotations

import json
import os
import subprocess
import sys
import time

import torch

PKG = os.path.dirname(os.path.abspath(__file__))
PROBE = os.path.join(PKG, "gemm_probe")

SHAPES = [
    ("logits (short k)", "ntt", 151808, 16384, 2048),
    ("logits (short k)", "nt8", 151808, 16384, 2048),
    ("logits (short k), 4 wavefronts", "nt4", 151808, 16384, 2048),
    ("dHidden (long k), 4 wavefronts", "nt4", 2048, 16384, 151936),
    ("dHidden (long k)", "nt8", 2048, 16384, 151936),
    ("dHidden (long k), untransposed weights", "mx4", 2048, 16384, 151936),
    ("dW (k-major operands)", "km8", 2048, 151808, 32768),
    ("dW (k-major operands)", "kmt", 2048, 151808, 32768),
    ("dW (k-major operands), 4 wavefronts", "km4", 2048, 151808, 32768),
    ("square", "nt8", 8192, 8192, 8192),
]


def vendor(label, variant, M, N, K, iters=4):
    dev = torch.device("cuda:0")
    if variant.startswith("km"):
        a = torch.randn(K, M, device=dev, dtype=torch.bfloat16)
        b = torch.randn(K, N, device=dev, dtype=torch.bfloat16)
        fn = lambda: a.T @ b
    else:
        a = torch.randn(M, K, device=dev, dtype=torch.bfloat16)
        b = torch.randn(N, K, device=dev, dtype=torch.bfloat16)
        fn = lambda: a @ b.T
    for _ in range(2):
        fn()
    torch.cuda.synchronize()
    t = time.perf_counter()
    for _ in range(iters):
        fn()
    torch.cuda.synchronize()
    dt = (time.perf_counter() - t) / iters
    return {"case": label, "variant": "torch.mm (vendor GEMM)", "M": M, "N": N, "K": K, "ms": dt * 1e3,
            "tflops": 2.0 * M * N * K / dt / 1e12}


def probe(label, variant, M, N, K):
    out = subprocess.run([PROBE, variant, str(M), str(N), str(K)], capture_output=True, text=True, timeout=600)
    if out.returncode != 0:
        raise RuntimeError(f"gemm_probe {variant} {M} {N} {K} failed: {out.stdout} {out.stderr}")
    rec = json.loads([l for l in out.stdout.splitlines() if l.startswith("{")][-1])
    rec["case"] = label
    rec["check"] = [l for l in out.stdout.splitlines() if "check" in l][-1]
    return rec


def main():
    if not torch.cuda.is_available():
        print("needs a GPU", file=sys.stderr)
        sys.exit(2)
    if not os.path.exists(PROBE):
        print(f"{PROBE} is missing: run python -m paper_2510_11062_amd.build", file=sys.stderr)
        sys.exit(2)
    for label, variant, M, N, K in SHAPES:
        print(json.dumps(probe(label, variant, M, N, K)), flush=True)
        if variant in ("nt8", "km8"):     # one vendor line per shape
            print(json.dumps(vendor(label, variant, M, N, K)), flush=True)


if __name__ == "__main__":
    main()
