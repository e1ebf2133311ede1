"""What the compiler makes of a kernel, where a small change of the source has cost a loop dearly: the kernel's own
assembly, compiled here."""
import re
import subprocess

import pytest

from paper_2104_09455_amd import build

SOURCE = """
#include "gemm_configs.h"
#include "gemm_fast.h"
namespace abft {{
template __global__ void gemm_fast_kernel<CfgOf<{dt}, {cfg}>::type, CfgOf<{dt}, {cfg}>::NSTAGE, {mode}, false, {conv}>(const GemmArgs);
}}
"""


def assembly(tmp_path, **instance):
    src, asm = tmp_path / "one.hip", tmp_path / "one.s"
    src.write_text(SOURCE.format(**instance))
    subprocess.run([build.HIPCC, *build.FLAGS, "-I", build.CSRC, "--cuda-device-only", "-S", str(src), "-o", str(asm)],
                   check=True, capture_output=True, timeout=300)
    return asm.read_text().splitlines()


# copies per k tile and wavefront: rows of A and B over eight rows and wavefronts
@pytest.mark.parametrize("cfg,copies", [("CFG_F128", 8), ("CFG_F128T", 8), ("CFG_F64T", 12), ("CFG_F256N", 6)])
def test_copies_of_a_convolution_s_k_tile_go_out_without_a_branch(cfg, copies, tmp_path):
    """Every lane's address of a copy is a select (its pixel, or zeros): no copy sits behind an exec-mask region of its
    own, so that between two such regions there are whole k tiles' copies."""
    runs = [0]
    for line in assembly(tmp_path, dt="DT_BF16", cfg=cfg, mode="MODE_NONE" if cfg == "CFG_F256N" else "MODE_THREAD", conv="true"):
        if re.match(r"\ts_(and|or|xor|andn2)_saveexec", line):
            runs.append(0)
        elif re.match(r"\tglobal_load_lds", line):
            runs[-1] += 1
    assert sum(runs) >= 2 * copies
    assert all(n % copies == 0 for n in runs), runs


@pytest.mark.parametrize("dt,cfg,mode", [("DT_I8", "CFG_F256W", "MODE_GLOBAL"), ("DT_F16", "CFG_F128", "MODE_GLOBAL"), ("DT_BF16", "CFG_F256N", "MODE_GLOBAL_FED")])
def test_copies_know_their_place_in_lds(dt, cfg, mode, tmp_path):
    """The place a copy writes to is an offset into LDS, not a pointer that is compared with null first."""
    lines = assembly(tmp_path, dt=dt, cfg=cfg, mode=mode, conv="false")
    assert any(re.match(r"\tglobal_load_lds", line) for line in lines)
    assert not any(re.match(r"\ts_cselect_b32 m0", line) for line in lines)
