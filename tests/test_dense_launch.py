"""The dense kernel's launcher refuses what its blocks cannot do: from the
sweep's inverses with more than 32 orbitals a block holds one inverse at a time
and needs the barriers of the Abar part before it takes the second.  Host only:
a launch without a GPU fails with another code than the refusal."""
import os
import subprocess

import pytest

from paper_2511_05222_amd import build, vmc

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "vmc_pipeline.hpp"
using namespace vmcx;
int main(int, char **argv) {
    // (nothing of it is read: the launch is refused, or finds no GPU)
    SysDev S{};
    S.n_occ = atoi(argv[1]);
    MeasBufs<TYPE> mb{};
    TYPE t;
    double d;
    if (argv[2][0] == '1') mb.kst = &t;
    if (argv[3][0] == '1') mb.ktil = &t;
    if (argv[4][0] == '1') mb.promote_key = &d;
    WalkerOut o{};
    DenseLayout L{};
    printf("%d\n", launch_dense<TYPE>(S, nullptr, mb, o, nullptr, L, 1, nullptr) == hipErrorInvalidValue);
    return 0;
}
"""


@pytest.mark.parametrize("typ", ["double", "float"])
def test_state_needs_abar(tmp_path, typ):
    lib = vmc.lib()._name
    (tmp_path / "m.hip").write_text(MAIN)
    exe = str(tmp_path / "m")
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-host-only", "-std=c++17",
                    "-DTYPE=" + typ, "-I", build.CSRC, "-I", os.path.join(build.ROOT, "include"),
                    str(tmp_path / "m.hip"), "-L" + os.path.dirname(lib), "-l:" + os.path.basename(lib),
                    "-Wl,-rpath," + os.path.dirname(lib), "-o", exe], check=True)

    def refused(n, state, ktil, key):
        env = dict(os.environ, HIP_VISIBLE_DEVICES="-1")   # no device, wherever this runs
        out = subprocess.run([exe, str(n), str(state), str(ktil), str(key)], check=True, capture_output=True, env=env,
                             text=True).stdout
        return out.strip() == "1"

    for n in (33, 48, 49, 64):
        assert refused(n, 1, 0, 0)
        assert not refused(n, 1, 1, 0) and not refused(n, 1, 0, 1) and not refused(n, 0, 0, 0)
    assert not refused(32, 1, 0, 0)
