"""Compile-time guard for the contraction kernels: no instantiation may spill registers (a spill inside the
tile loop once halved the wide-row kernel's speed without failing any numerical test).  Uses hipcc's resource-usage remarks; no GPU needed."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not (os.path.exists(HIPCC) or shutil.which("hipcc")), reason="hipcc not available")
def test_dot_product_contraction_kernels_do_not_spill(tmp_path):
    """fp32 matrix instructions (TransE; small evaluations of the others): rows copied straight to LDS or through registers."""
    src = os.path.join(ROOT, "paper_2101_08358_amd", "csrc", "mar_flash.hip")
    cmd = [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-Rpass-analysis=kernel-resource-usage", "-c", src, "-o", str(tmp_path / "flash.o")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    blocks = re.split(r"remark: Function Name: ", r.stderr)[1:]
    seen = {"forward, registers": 0, "forward, direct": 0, "backward": 0}
    for b in blocks:
        name = b.split()[0]
        kind = re.match(r"_Z(7k_flash|11k_flash_bwd)I(?:Li\d+E)*Li(\d+)EEv9FlashArgs$", name)
        if not kind:
            continue
        # the forward kernel's last template argument: 1 = tiles copied straight to LDS
        seen["backward" if "bwd" in name else ("forward, registers", "forward, direct")[int(kind.group(2))]] += 1
        spill = int(re.search(r"VGPRs Spill: (\d+)", b).group(1))
        scratch = int(re.search(r"ScratchSize \[bytes/lane\]: (\d+)", b).group(1))
        assert spill == 0 and scratch == 0, (name, spill, scratch)
    assert seen == {"forward, registers": 15, "forward, direct": 9, "backward": 5}, seen


@pytest.mark.skipif(not (os.path.exists(HIPCC) or shutil.which("hipcc")), reason="hipcc not available")
def test_split_precision_kernels_do_not_spill(tmp_path):
    src = os.path.join(ROOT, "paper_2101_08358_amd", "csrc", "mar_split.hip")
    cmd = [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-Rpass-analysis=kernel-resource-usage", "-c", src, "-o", str(tmp_path / "split.o")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    blocks = re.split(r"remark: Function Name: ", r.stderr)[1:]
    seen = {"k_split": 0, "k_split_carry": 0, "k_split_dist": 0}
    for b in blocks:
        name = b.split()[0]
        kind = re.match(r"_Z\d+(k_split|k_split_carry|k_split_dist)I", name)
        if not kind:
            continue
        seen[kind.group(1)] += 1
        spill = int(re.search(r"VGPRs Spill: (\d+)", b).group(1))
        scratch = int(re.search(r"ScratchSize \[bytes/lane\]: (\d+)", b).group(1))
        assert spill == 0 and scratch == 0, (name, spill, scratch)
    # eight widths; two passes in either precision and evaluation; the passes with pieces of the row order; TransE's with and without
    assert seen == {"k_split": 8 * 5, "k_split_carry": 8 * 4, "k_split_dist": 8 * 4}, seen


@pytest.mark.skipif(not (os.path.exists(HIPCC) or shutil.which("hipcc")), reason="hipcc not available")
def test_narrow_evaluation_exchanges_nothing_between_lanes(tmp_path):
    """Rows up to 96 floats, and from 105 to 112: a tile's comparisons take as long as its products, so the scores come out of the
    matrix pipe in the lanes that compare them (an exchange after 16 x 16 blocks made such evaluations 2 to 10% slower)."""
    src = os.path.join(ROOT, "paper_2101_08358_amd", "csrc", "mar_split.hip")
    cmd = [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-Rpass-analysis=kernel-resource-usage", "--offload-device-only", "-S", src, "-o", str(tmp_path / "split.s")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    text = (tmp_path / "split.s").read_text()
    bodies = {(m.group(1), int(m.group(2))): m.group(3)
              for m in re.finditer(r"^_Z\d+(k_split|k_split_eval_full)ILi(\d+)E(?:Li3ELb1E)?Ev9FlashArgs:(.*?)^\.Lfunc_end", text, re.S | re.M)}
    assert sorted(bodies) == [("k_split", nk) for nk in (2, 4, 6, 7, 8, 12, 16, 25)] + [("k_split_eval_full", 7)]
    for kernel in (("k_split", 2), ("k_split", 4), ("k_split", 6), ("k_split_eval_full", 7)):
        assert "permlane16_swap" not in bodies[kernel], kernel
        assert bodies[kernel].count("v_mfma_f32_32x32x16_f16") == 3 * kernel[1], kernel
    full = [b for b in re.split(r"remark: Function Name: ", r.stderr)[1:] if "k_split_eval_full" in b.split()[0]]
    assert len(full) == 1 and re.search(r"VGPRs Spill: 0\b", full[0]) and re.search(r"ScratchSize \[bytes/lane\]: 0\b", full[0])
