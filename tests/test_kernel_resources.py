"""Register budget of the kernels (CPU only: a compile, no launch).

The persistent GEMM and the split-K G^ kernels run one wave per SIMD and keep their
accumulators in the accumulation registers; the tile, direct G^, fp32 and decompression
kernels and the row kernels of the block keep accumulators, fragments or whole rows in
registers through fully unrolled loops.  Any VGPR spill or private (scratch) array inside
them turns into scratch-memory traffic whose waits share the vector-memory counter with
the operand copies, and each such wait drains every copy in flight.  The units are
compiled as build.py compiles them, with the compiler's resource-usage remarks, and every
kernel listed must use no scratch memory and spill no VGPR.

The G^ kernels read their fragments by inline assembly that the compiler takes as
finished at once; the generated code must leave the registers of such a read alone until
the wait that follows it."""
import functools
import os
import re
import subprocess
import sys
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@functools.lru_cache(maxsize=None)
def _compile(unit):
    """The remarks of every kernel of the unit, and its device assembly."""
    sys.path.insert(0, ROOT)
    from paper_2410_15352_amd import build as B
    try:
        hipcc = B.hipcc()
    except RuntimeError:
        pytest.skip("hipcc not available")
    extra = dict(B.UNITS)[unit]
    with tempfile.TemporaryDirectory(prefix="compact_res_") as d:
        out = os.path.join(d, "u.s")
        cmd = [hipcc, *B.FLAGS, *extra, "-I", B.INCLUDE, "--offload-device-only", "-S", os.path.join(B.CSRC, unit),
               "-o", out, "-Rpass-analysis=kernel-resource-usage"]
        res = subprocess.run(cmd, capture_output=True, text=True, cwd=d)
        assert res.returncode == 0, res.stderr[-2000:]
        with open(out) as f:
            asm = f.read()
    kernels, cur = {}, None
    for line in res.stderr.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            cur = m.group(1)
            kernels[cur] = {}
            continue
        m = re.search(r"remark:\s+([A-Za-z ]+?)(?: \[[^\]]*\])?: (\d+) \[", line)
        if m and cur is not None:
            kernels[cur][m.group(1).strip()] = int(m.group(2))
    return kernels, asm


# unit -> kernels and how many instantiations of each
KERNELS = {
    "kernels_w4.hip": {"k_gemm_w4": 16, "k_ghat_w4": 3, "k_dec_w4": 6, "k_ghat_direct": 1},
    "kernels_tile.hip": {"k_gemm_tile": 8},
    "compact_api.hip": {"k_fwd_f32": 2, "k_bwd_f32": 2, "k_dec_f32": 3, "k_adam_pt_batched": 3},
    "block_ops.hip": {"k_rmsnorm_fwd": 8, "k_rmsnorm_bwd": 12, "k_swiglu_": 2, "k_ce_": 3, "k_join3": 1},
}


@pytest.mark.parametrize("unit", list(KERNELS))
def test_persistent_kernels_use_no_scratch(unit):
    kernels, _ = _compile(unit)
    for name, count in KERNELS[unit].items():
        found = [k for k in kernels if name in k]
        assert len(found) == count, (name, sorted(kernels))
        for k in found:
            r = kernels[k]
            assert r.get("ScratchSize") == 0, (k, r)
            assert r.get("VGPRs Spill") == 0, (k, r)


def test_occupancy_the_launch_bounds_promise():
    """Waves per SIMD: two for the tile kernels' eight waves and the fp32 ones, four for the
    decompression of bf16 weights (four workgroups per CU)."""
    for unit, name, least in (("kernels_tile.hip", "k_gemm_tile", 2), ("compact_api.hip", "_f32ILb", 2),
                              ("compact_api.hip", "k_dec_f32", 2), ("kernels_w4.hip", "k_dec_w4ILb0", 4)):
        for k, r in _compile(unit)[0].items():
            if name in k:
                assert r["Occupancy"] >= least, (k, r)


def _registers(text):
    """Numbers of the vector registers that an instruction names."""
    out = set()
    for lo, hi, one in re.findall(r"\bv(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
        out.update([int(one)] if one else range(int(lo), int(hi) + 1))
    return out


def test_transposing_reads_are_left_alone_until_their_wait():
    _, asm = _compile("kernels_w4.hip")
    reads = 0
    for body in re.split(r"^(?=_ZN7compact\S+:)", asm, flags=re.M):
        if not re.match(r"_ZN7compact\d+k_ghat_", body):
            continue
        pending = set()
        for line in body.split(".Lfunc_end")[0].splitlines():
            ins = line.split(";")[0].strip()
            if not ins or ins.startswith(".") or ins.endswith(":"):
                continue
            if re.match(r"s_waitcnt\b.*lgkmcnt\(0\)", ins):
                pending = set()
                continue
            touched = _registers(ins) & pending
            assert not touched, f"{ins}: v{sorted(touched)} still being read into"
            if ins.startswith("ds_read_b64_tr_b16"):
                reads += 1
                pending |= _registers(ins.split(",")[0])
    assert reads >= 64
