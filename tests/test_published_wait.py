"""Partial results that workgroups of one launch exchange have to be in memory before the ticket that
announces them is taken: between the stores and the ticket's atomic the code must wait for the stores.
(A workgroup-scope release fence in the place of all_published() compiles to no such wait.)"""
import os
import re
import subprocess

import pytest

from conftest import ROOT

SRC = r'''
#include <hip/hip_runtime.h>
#include "lt_reduce.h"
__global__ void exchange(float* parts, uint32_t* ticket, float4 v) {
  if (threadIdx.x < 64u) {
    ltk::publish4(parts + (blockIdx.x * 64u + threadIdx.x) * 4u, v);
    WAIT;
  }
  __syncthreads();
  if (threadIdx.x == 0u) atomicAdd(ticket, 1u);
}
'''


def waits(tmp_path, wait):
    src, out = tmp_path / "x.hip", tmp_path / "x.s"
    src.write_text(SRC.replace("WAIT", wait))
    hipcc = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("needs hipcc")
    r = subprocess.run([hipcc, "-O3", "-std=c++17", "--offload-arch=gfx950", "-S", "--cuda-device-only", "-I" + os.path.join(ROOT, "paper_2102_13267_amd", "csrc"),
                        str(src), "-o", str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    lines = out.read_text().splitlines()
    stores = [i for i, l in enumerate(lines) if re.search(r"global_store\S* .*sc1", l)]
    atomic = next(i for i, l in enumerate(lines) if "global_atomic_add" in l)
    assert stores and max(stores) < atomic
    return any(re.search(r"s_waitcnt.*vmcnt\(0\)", l) for l in lines[max(stores):atomic])


def test_stores_are_waited_for_before_the_ticket(tmp_path):
    assert waits(tmp_path, "ltk::all_published()")
    assert not waits(tmp_path, "")                       # (the check itself sees a missing wait)


def test_every_exchange_waits():
    """Every kernel that publishes partial results calls all_published() before its ticket."""
    csrc = os.path.join(ROOT, "paper_2102_13267_amd", "csrc")
    for f in sorted(os.listdir(csrc)):
        if not f.endswith(".hip"):
            continue
        text = open(os.path.join(csrc, f)).read()
        for m in re.finditer(r"atomicAdd\(", text):
            before = text[:m.start()]
            assert before.rfind("all_published();") > max(before.rfind("publish("), before.rfind("publish4(")), (f, text[m.start():m.start() + 60])
