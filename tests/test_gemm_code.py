"""What the compiler makes of the GEMM's assembly blocks (compiled for gfx950 here, nothing is run)."""
import os
import re
import shutil
import subprocess

from paper_2602_08387_amd import build as b

HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

# one block of MFMAs, and its results rounded and stored: the conversions need nothing but the accumulators
DRAIN = """
#include "gemm_core.h"
using namespace dl;
__global__ __launch_bounds__(512) void drained(const bf16x8* in, bf16_t* out, int n) {
  f32x4 acc[2][4];
  for (int i = 0; i < 2; ++i)
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0, 0, 0, 0};
  const int l = threadIdx.x;
  for (int k = 0; k < n; ++k) {
    const bf16x8* p = in + (size_t)k * 512 * 12 + l;
    mfma_quadrant(acc[0][0], acc[1][0], acc[0][1], acc[1][1], acc[0][2], acc[1][2], acc[0][3], acc[1][3], p[0], p[512], p[1024], p[1536],
                  p[2048], p[2560], p[3072], p[3584], p[4096], p[4608], p[5120], p[5632]);
  }
  mfma_drain(acc);
  for (int i = 0; i < 2; ++i)
    for (int j = 0; j < 4; ++j)
      for (int e = 0; e < 4; ++e) out[((i * 4 + j) * 4 + e) * 512 + l] = (bf16_t)acc[i][j][e];
}
"""


def _compile(tmp_path, *args):
    r = subprocess.run([HIPCC, *b.FLAGS, "-I", b.CSRC, "--offload-device-only", *args], capture_output=True, text=True, cwd=tmp_path)
    assert r.returncode == 0, r.stderr[-3000:]
    return r.stderr


def test_no_accumulator_is_read_before_the_last_mfma_has_written_it(tmp_path):
    """The MFMAs are assembly, so the compiler knows of no hazard: only the dependence on mfma_drain() keeps it from converting an
    accumulator right behind them."""
    (tmp_path / "drain.hip").write_text(DRAIN)
    _compile(tmp_path, "-S", "drain.hip", "-o", "drain.s")
    ops = [m[1] for m in re.finditer(r"^\s+([vs]_\w+)(?: 15\b)?", (tmp_path / "drain.s").read_text(), re.M)
           if m[1].startswith(("v_mfma", "v_cvt")) or m[0].rstrip().endswith("s_nop 15")]
    last_mfma = max(i for i, op in enumerate(ops) if op.startswith("v_mfma"))
    behind = ops[last_mfma + 1:]
    assert behind[0] == "s_nop" and sum(op.startswith("v_cvt") for op in behind) >= 16, behind


def test_the_persistent_kernels_spill_no_vector_register_and_store_what_their_waits_count(tmp_path):
    """The reload of a spilled register is counted in order behind the next tile's loads and the last tile's stores: whatever
    waits for it waits for all of those.  And the wait for the next tile's loads counts a wave's stores of a tile inside C, 16 or, with
    two or three outputs, 32: fewer would leave loads unwaited for."""
    out = _compile(tmp_path, "-Rpass-analysis=kernel-resource-usage", "-S", os.path.join(b.CSRC, "gemm.hip"), "-o", "gemm.s")
    spills = {}
    for m in re.finditer(r"(Function Name|VGPRs Spill|ScratchSize \[bytes/lane\]): (\S+)", out):
        if m[1] == "Function Name":
            name = m[2]
        else:
            spills[name] = spills.get(name, 0) + int(m[2])
    assert len(spills) == 14 and all("gemm" in n for n in spills), spills
    assert not any(spills.values()), spills
    text = (tmp_path / "gemm.s").read_text()
    for name in spills:
        code = text[text.index(f"\n{name}:"):]
        stores = len(re.findall(r"^\s+(?:global|flat|buffer)_store", code[:code.index(".Lfunc_end")], re.M))
        assert stores == (32 if "swiglu" in name else 16), (name, stores)


def test_the_one_tile_kernels_ask_for_the_whole_residual_before_they_wait(tmp_path):
    """The tile's residual (or old value) is requested in three to eight loads per thread behind each other; a wait between two of them
    made products of few K-steps up to 16 % slower."""
    _compile(tmp_path, "-S", os.path.join(b.CSRC, "gemm_tile.hip"), "-o", "tile.s")
    text = (tmp_path / "tile.s").read_text()
    kernels = re.findall(r"^(_ZN2dl\d+gemm_tile(?:_group)?_kernel\w*Li0EEE\w+):", text, re.M)
    assert len(kernels) == 15, kernels
    for name in kernels:
        code = text[text.index(f"\n{name}:"):]
        ops = re.findall(r"global_load_dwordx4|s_waitcnt [^\n]*vmcnt", code[:code.index(".Lfunc_end")])
        first, last = ops.index("global_load_dwordx4"), len(ops) - 1 - ops[::-1].index("global_load_dwordx4")
        assert all(op == "global_load_dwordx4" for op in ops[first:last]), (name, ops[first:last])
