"""LDS accesses of the passes that one wavefront runs without barriers, in the
device code the compiler forms: lanes read what others wrote, so a load must
not be passed by a later store, nor a store by a later load.  A fence holds
them, and a store whose value depends on the load cannot pass it anyway."""
import re
import subprocess

from paper_2202_11288_amd import build as BLD

PASSES = """#include "fourstep.hpp"
namespace amg {
#define ROWS(T, SYM)                                                                           \\
  template __global__ void k_row<T, true, SYM, 7>(LevelDev<T>, cplx<T>*, Twiddles<T>, const T*, \\
                                                  int, const T*);                              \\
  template __global__ void k_row<T, true, SYM, 8>(LevelDev<T>, cplx<T>*, Twiddles<T>, const T*, \\
                                                  int, const T*);
#define COLS(T, LOG2)                                                                          \\
  template __global__ void k_col_fwd<T, COL_MV, ColGeom<LOG2, 2>>(LevelDev<T>, ColIn<T>,       \\
                                                                  cplx<T>*, Twiddles<T>, T*);  \\
  template __global__ void k_col_inv<T, EPI_MV, ColGeom<LOG2, 2>>(                             \\
      LevelDev<T>, EpiOut<T>, const cplx<T>*, Twiddles<T>, double*);
ROWS(double, true) ROWS(double, false) ROWS(float, true) ROWS(float, false)
COLS(double, 6) COLS(double, 7) COLS(float, 6) COLS(float, 7)
}
"""


def violations(body):
    """Pairs (load, store) that only the compiler's choice keeps in order, in the
    text behind the first wavefront fence (nothing is read from LDS before it)."""
    deps, loads, bad, half = {}, [], 0, None
    stored = started = False
    for line in body.splitlines():
        if " fence " in line:
            started = started or 'syncscope("wavefront")' in line
            loads, stored, half = [], False, None
            continue
        names = re.findall(r"%[\w.]+", line)
        d = re.match(r"\s+(%[\w.]+) = (?:tail )?(\w+)", line)
        if d:
            if d.group(2) == "load":
                lds = "addrspace(3)" in line and started
                bad += lds and stored
                loads += [d.group(1)] if lds else []
                deps[d.group(1)] = {d.group(1)} if lds else set()
            else:
                deps[d.group(1)] = set().union(*(deps.get(n, set()) for n in names[1:]))
        elif re.match(r"\s+store ", line) and "addrspace(3)" in line and started:
            value = line.split("ptr addrspace(3)")[0]
            have = set().union(*(deps.get(n, set()) for n in re.findall(r"%[\w.]+", value)))
            stored = True
            if half is None:  # the two halves of a complex value never meet in a slot
                half = have
                continue
            bad += len(set(loads) - (half | have))
            half = None
    return bad


def test_lane_exchanges_are_ordered(tmp_path):
    src, ll = tmp_path / "passes.hip", tmp_path / "passes.ll"
    src.write_text(PASSES)
    cmd = [BLD.hipcc()] + BLD.COMMON + ["-x", "hip"] + BLD.DEVICE + [
        "--offload-device-only", "-S", "-emit-llvm", "-I" + BLD.CSRC, str(src), "-o", str(ll)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    kernels = re.findall(r"^define [^\n]*amdgpu_kernel void @(\S+?)\((.*?)^}", ll.read_text(),
                         re.S | re.M)
    assert len(kernels) == 16
    assert {name: violations(body) for name, body in kernels} == {name: 0 for name, _ in kernels}
    for name, body in kernels:
        assert len(re.findall("llvm.amdgcn.wave.barrier", body)) >= 1, name
