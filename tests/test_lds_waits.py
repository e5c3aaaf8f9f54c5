"""Waits that order LDS writes.  The convolution kernels that hold a tile's pixels in LDS: every wave waits for its own part of the filters before a
barrier behind which others read it, also a wave that stages no pixel because the tile has few of them.  The kernel of uint8 codes: flip flags are
cleared before the loads that bring them in are sent."""
import os
import re
import subprocess

import pytest
import torch


def _kernels(source, tmp_path):
    """The instructions of every kernel of a source file, as hipcc compiles it."""
    from paper_1609_07061_amd import build

    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    out = str(tmp_path / "kernels.s")
    subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, source), "-o", out], check=True, capture_output=True)
    kernels, code = {}, None
    for line in open(out):
        line = line.split(";")[0].strip()
        label = re.fullmatch(r"(_Z\w+):", line)
        if label:
            code = kernels.setdefault(label.group(1), [])
        elif line and code is not None and not line.startswith(".") and not line.endswith(":"):
            code.append(line)
    return {name: code for name, code in kernels.items() if any(i.startswith("s_endpgm") for i in code)}


def test_barriers_count_loads(tmp_path):
    kernels = _kernels("qnn_gemm_image.hip", tmp_path)
    assert len(kernels) == 6
    for name, code in kernels.items():
        waits = [code[i - 1] for i, instruction in enumerate(code) if instruction.startswith("s_barrier")]
        assert waits and all(re.match(r"s_waitcnt vmcnt\(\d+\) lgkmcnt\(0\)", w) for w in waits), (name, waits)


def test_flags_are_cleared_before_they_arrive(tmp_path):
    kernels = {name: code for name, code in _kernels("qnn_gemm_codes.hip", tmp_path).items() if "gemm_codes_kernel" in name}
    assert len(kernels) == 2
    for name, code in kernels.items():
        cleared = min(i for i, instruction in enumerate(code) if instruction.startswith("ds_write"))
        sent = min(i for i, instruction in enumerate(code) if instruction.startswith("global_load_lds_"))
        assert cleared < sent and any(re.match(r"s_waitcnt.*lgkmcnt\(0\)", i) for i in code[cleared:sent] if "vmcnt" not in i), name


@pytest.mark.gpu
@pytest.mark.parametrize("B,H,W,C,N", [
    (64, 16, 16, 64, 128),   # 171 LDS pixels of one piece in every tile: one wave has none
    (256, 8, 8, 128, 100),   # 172, two images a tile
    (129, 12, 12, 32, 128),  # last tile of 16 pixels: 53 in LDS
    (37, 28, 28, 64, 130),   # ... of 80 pixels: 146
])
@pytest.mark.parametrize("bits", [1, 2, 4])
def test_waves_without_pixels(seed, B, H, W, C, N, bits):
    import paper_1609_07061_amd as q
    from qnn_testlib import kernels_of
    from test_gpu_image import _operands

    torch.manual_seed(seed)
    planes, w, want = _operands(q, B, H, W, C, N, bits)
    coef = [1 << p for p in range(bits)]
    call = lambda: q.qnn_bitplane_conv2d(planes, coef, q.PLANE_BIT, C, w, [1], q.PLANE_SIGN, 1, 1)
    assert torch.equal(call().to(torch.int64), want)
    assert all(k.startswith("gemm_image_kernel") for k in kernels_of(call))
    T = torch.zeros(N, dtype=torch.int32, device="cuda")
    got = q.qnn_bitplane_conv2d_sign(planes, coef, q.PLANE_BIT, C, w, [1], q.PLANE_SIGN, 1, 1, T)
    assert torch.equal(got, q.qnn_pack_sign(want.reshape(-1, N).float()).reshape(got.shape))
