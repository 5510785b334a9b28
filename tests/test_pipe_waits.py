"""The register-tile pipeline's epilogue parameters are written to LDS by one wave and read by all:
between the write and the workgroup's next meeting the writing wave must wait for its LDS operations,
whatever the number of K chunks.  Checked in the gfx950 assembly of the kernels built here, since a
missing wait shows on the device only by timing."""
import re
import subprocess

import pytest

from paper_2307_04339_amd import build

# tile_m, tile_n, waves along m: three operand reads ahead (64 wide) and one
KERNELS = [(64, 64, 2), (128, 64, 4), (128, 128, 2)]

SOURCE = """#include "gemm_pipe.h"
namespace miriam {
%s
}
"""


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    d = tmp_path_factory.mktemp("pipe_waits")
    inst = [f"template __global__ void pipe_kernel<bf16_t, {tm}, {tn}, {wm}, {p}, {taps}, {nb}>(IgemmArgs, Shard);"
            for tm, tn, wm in KERNELS for p in (2, 4) for taps, nb in [("false", "false"), ("true", "false"), ("false", "true")]
            if nb == "false" or tn == 64]
    src, out = d / "waits.hip", d / "waits.s"
    src.write_text(SOURCE % "\n".join(inst))
    r = subprocess.run(["hipcc", *build.FLAGS, f"-I{build.CSRC}", "-S", "--cuda-device-only", "-o", str(out), str(src)],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    kernels = re.findall(r"^(_ZN6miriam11pipe_kernel\w+):\s.*?\n(.*?)^\.Lfunc_end", out.read_text(), re.S | re.M)
    assert len(kernels) == len(inst), [k for k, _ in kernels]
    return kernels


def test_parameter_writes_are_waited_for_before_the_next_meeting(assembly):
    for name, body in assembly:
        writes = pending = 0
        for line in body.splitlines():
            op = line.split(";")[0].strip()
            if op.startswith("ds_write"):
                writes += 1
                pending = 1
            elif op.startswith("s_waitcnt") and "lgkmcnt(0)" in op:
                pending = 0
            elif op.startswith("s_barrier"):
                assert not pending, f"{name}: a meeting with the parameter write outstanding"
        assert writes, f"{name}: no parameter write found"
