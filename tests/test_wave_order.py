"""Lanes of the spreading's wavefronts clear LDS records that other lanes fill next.
The compiler's intermediate code has to keep that order: after the last store of
Octants::clear come a release and an acquire fence of wavefront scope."""
import re
import subprocess

from paper_2408_14140_amd import build as B

KERNEL = """
#include "octants.h"
using namespace ibx;
__global__ void use(float* out)
{
    __shared__ Octants<float, 4, false>::Lds mem;
    Octants<float, 4, false> oct(mem);
    oct.clear();
    out[threadIdx.x] = mem.rec[threadIdx.x];
}
"""


def _function(ir, name):
    """Text of the function whose (mangled) name contains `name`."""
    for body in re.findall(r"^define [^\n]*\{\n.*?^\}", ir, re.M | re.S):
        if name in body.split("\n", 1)[0]:
            return body
    raise AssertionError(f"no function {name}")


def test_clearing_records_is_ordered_before_filling_them(tmp_path):
    src, out = tmp_path / "use.hip", tmp_path / "use.ll"
    src.write_text(KERNEL)
    flags = [f if f != "-O3" else "-O1" for f in B.FLAGS]
    subprocess.run([B.HIPCC] + flags + ["--offload-device-only", "-S", "-emit-llvm", "-Xclang",
                                        "-disable-llvm-passes", "-o", str(out), str(src)],
                   check=True, stderr=subprocess.DEVNULL)
    ir = out.read_text()
    clear = _function(ir, "5clearEv")
    last = clear[clear.rindex("store "):]
    call = re.search(r"call void @(\w*10wave_order\w*)\(", last)
    assert call, "nothing orders the stores of clear()"
    order = _function(ir, call.group(1))
    fences = re.findall(r'fence syncscope\("wavefront"\) (\w+)', order)
    assert fences == ["release", "acquire"]
