"""The broadcast and resident kernels' loops of stores, in the code the compiler
makes of them: a loop that stores a loaded value to one destination after
another must not wait for memory (s_waitcnt vmcnt), which would send each store
out a round trip after the one before it.  Only the kernels that pace their
stores on purpose may."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1511_00175_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def kernels(text):
    """(name, lines) of every kernel of a listing."""
    name, body = None, []
    for line in text.splitlines():
        m = re.match(r"(_ZN\S+):", line)
        if m:
            name, body = m[1], []
        elif name:
            body.append(line)
            if "s_endpgm" in line:
                yield name, body
                name = None


def waiting_loops(body):
    """Labels of the loops that store, load nothing and wait for memory."""
    label = {m[1]: i for i, line in enumerate(body) if (m := re.match(r"(\.LBB\S+?):", line))}
    out = []
    for i, line in enumerate(body):
        m = re.search(r"s_c?branch\S*\s+(\.LBB\S+)", line)
        if m and label.get(m[1], i) < i:
            loop = "\n".join(body[label[m[1]]:i + 1])
            if "buffer_store" in loop and not re.search(r"(buffer|global|flat)_load", loop) and "vmcnt" in loop:
                out.append(m[1])
    return out


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    """The code of a source file, compiled once."""
    if not os.path.exists(HIPCC):
        pytest.skip("needs hipcc")
    made = {}

    def compile_one(src):
        if src not in made:
            asm = tmp_path_factory.mktemp("asm") / "out.s"
            cmd = [HIPCC, "-O3", "-std=c++17", "--offload-arch=gfx950", "-ffp-contract=off",
                   "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", f"-I{os.path.join(ROOT, 'include')}",
                   f"-I{CSRC}", "--cuda-device-only", "-S", "-o", str(asm), os.path.join(CSRC, src)]
            r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
            assert r.returncode == 0, r.stderr
            made[src] = list(kernels(asm.read_text()))
        return made[src]

    return compile_one


def test_broadcast_stores_do_not_wait(listing):
    seen = [(name, waiting_loops(body)) for name, body in listing("fc_update.hip") if "bcast_kernel" in name]
    assert len(seen) >= 5
    paced = [name for name, loops in seen if "bcast_kernelILi4ELi1ELi1E" in name]
    assert {name: loops for name, loops in seen if loops and name not in paced} == {}


@pytest.mark.parametrize("src", ["fc_reduce_f32.hip", "fc_reduce_f16.hip"])
def test_resident_stores_do_not_wait(listing, src):
    """The resident kernels store what lies in LDS, copies of w' included, and
    their replicas were all read before."""
    seen = [(name, waiting_loops(body)) for name, body in listing(src) if "resident_kernel" in name]
    assert len(seen) >= 20
    assert {name: loops for name, loops in seen if loops} == {}


@pytest.mark.parametrize("src", ["fc_reduce_f32.hip", "fc_reduce_f16.hip"])
def test_resident_tiles_of_few_read_descriptors_one_by_one(listing, src):
    """Resident kernels without register-held tiles serve plans whose waves may
    have one tile: they read a tile's descriptor with a scalar load, not with a
    vector load for the round, whose longer wait comes before the first
    replica (replicas, w and v are read with buffer loads)."""
    few = [(name, [x for x in body if "global_load_dwordx4" in x]) for name, body in listing(src)
           if "resident_kernel" in name and name.split("EEEv")[0].endswith("ELi0")]
    assert len(few) >= 12
    assert {name: loads for name, loads in few if loads} == {}
