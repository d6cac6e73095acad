"""Where the lanes of a wave exchange values through LDS (stores in column
order, the resampler's rows), the writes, the reads and the next writes are
ordered for the compiler as well: a fence of the wave on both sides of the
reads, in the code handed to the optimiser."""
import re
import subprocess

import pytest

from paper_2312_00229_amd import build


def functions(source, *macros):
    """{name: calls and fences in order} of a source's device code before any optimisation."""
    try:
        hipcc = build.hipcc()
    except RuntimeError as e:
        pytest.skip(str(e))
    text = subprocess.run([hipcc, "-O3", *build.DEVICE_FLAGS, *macros, "--offload-device-only", "-S", "-emit-llvm",
                           "-Xclang", "-disable-llvm-passes", "%s/%s" % (build.CSRC, source), "-o", "-"],
                          check=True, capture_output=True, text=True).stdout
    found = {}
    for body in re.findall(r"^define .*?^}", text, flags=re.S | re.M):
        name = re.search(r"@(\w+)\(", body)[1]
        found[name] = re.findall(r"call [^@]*@([\w.]+)\(|(fence syncscope\(\"wavefront\"\) \w+)", body)
        found[name] = [a or b for a, b in found[name]]
    return found


def check_orders(funcs, names, stores):
    assert names
    for name in names:
        marks = [{"_ZN2wz14wave_lds_orderEv": "order"}.get(c, "store") for c in funcs[name]
                 if c == "_ZN2wz14wave_lds_orderEv" or re.search(stores, c)]
        assert marks[0] == marks[-1] == "order" and len(marks) > 2 and set(marks[1:-1]) == {"store"}, (name, marks)


def test_the_fence():
    funcs = functions("weno_zoom.hip", "-DWENO_IO=2")
    assert funcs["_ZN2wz14wave_lds_orderEv"] == ['fence syncscope("wavefront") release', "llvm.amdgcn.wave.barrier",
                                                 'fence syncscope("wavefront") acquire']


@pytest.mark.parametrize("io", [2, 3])
def test_staged_stores(io):
    funcs = functions("weno_zoom.hip", "-DWENO_IO=%d" % io)
    # one and two columns per lane
    check_orders(funcs, [f for c in (1, 2) for f in funcs if "11store_quadsILi%dELi%dE" % (c, io) in f], "buf_st_f32")


def test_resampled_rows():
    funcs = functions("weno_resample.hip")
    # the row step of every wave kernel: 2 beta modes x 4 row lengths x 4 pairs of types
    names = [f for f in funcs if "wave_resample_kernel" in f and any("interval_value" in c for c in funcs[f])
             and any("buf_st_" in c for c in funcs[f])]
    assert len(names) == 32
    check_orders(funcs, names, "buf_st_")
