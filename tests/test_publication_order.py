"""A reduction without counters (once_sum) rests on every wave's reads being issued after its own words have reached
memory.  Nothing in the data says so, so the order has to be one that the compiler must keep: checked in its
intermediate form and in the instructions it emits."""
import os
import re
import subprocess

import pytest

from paper_2605_12245_amd import build

SOURCE = """
#include <hip/hip_runtime.h>
#include <cstdint>
#include "soar.h"
#include "soar_once.hpp"
extern "C" __global__ void reduce_once(uint64_t *words, uint64_t *epoch, uint64_t nonce, uint32_t G, double *sum)
{
    double v = (double)blockIdx.x;
    bool flag = false;
    if (once_sum(words, epoch, 7u, nonce, blockIdx.x, G, v, flag)) *sum = v;
}
"""


def emitted(tmp_path, *how):
    src, out = tmp_path / "reduce.hip", tmp_path / "reduce.out"
    src.write_text(SOURCE)
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC", "-Wall")]
    cmd = [build.HIPCC, *flags, "-w", "-I", os.path.join(build.HERE, "csrc"), "--cuda-device-only", "-S", *how, str(src), "-o", str(out)]
    subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    text = out.read_text()
    return text[text.index("reduce_once"):].splitlines()


@pytest.mark.parametrize("form", ["intermediate", "assembly"])
def test_words_are_read_after_the_own_ones_have_been_performed(tmp_path, form):
    if form == "assembly":
        lines = emitted(tmp_path)
        store, load, wait = (re.compile(p) for p in (r"\bglobal_store_dwordx2|\bflat_store_dwordx2", r"\b(global|flat)_load_dwordx2.* sc1",
                                                     r"\bs_waitcnt vmcnt\(0\)"))
    else:
        lines = emitted(tmp_path, "-emit-llvm")
        store, load, wait = (re.compile(p) for p in (r"store atomic i64", r"load atomic i64", r"asm sideeffect \"s_waitcnt vmcnt\(0\).*~\{memory\}"))
    loads = [k for k, l in enumerate(lines) if load.search(l)]
    assert loads
    stores = [k for k, l in enumerate(lines) if store.search(l) and k < loads[0]]
    assert stores, "nothing is published before the first read"
    assert any(wait.search(l) for l in lines[stores[-1] + 1:loads[0]]), "nothing holds the reads back"
