"""The checks of test_generated_code.py on the kernels that stream weights through rings in LDS: their direct loads are issued and awaited by
hand too, so the compiler knows nothing of their scalar bases, of M0 and of what is in flight."""
import functools
import os
import subprocess

import pytest

import test_generated_code as G
from paper_2604_00785_amd import binding as B

NAMES = ("stream_fwd_kernel", "route_gate_up_kernel", "down_combine_kernel")


@functools.lru_cache(None)
def kernels():
    B.load()
    found = {}
    for i, obj in enumerate(G._code_objects(B.LIB_PATH)):
        path = "/tmp/moe_stream_code_%d_%d.o" % (os.getpid(), i)
        with open(path, "wb") as f:
            f.write(obj)
        out = subprocess.run([G.OBJDUMP, "-d", "--no-show-raw-insn", path], capture_output=True, text=True, check=True).stdout
        os.remove(path)
        found.update({n: G.Kernel(code) for n, code in G._parse(out).items() if any(s in n for s in NAMES)})
    return found


@pytest.mark.parametrize("check", [G.base, G.in_flight, G.m0, G.settled], ids=lambda c: c.__name__)
def test_streaming_products(check):
    assert all(any(s in n for n in kernels()) for s in NAMES)
    for name, k in kernels().items():
        assert any(o.startswith("v_mfma") for o in k.op) and any(o.startswith("global_load_lds") for o in k.op), name
        bad = check(k)
        assert not bad, (name, len(bad), bad[:4])

