"""The tensor quantizer's per-channel scheme on either side of every rule on rows and columns: lane groups of 16, 32 and 64 per row,
ragged rows, row counts that end inside a wavefront's set."""
import numpy as np
import pytest
import torch

import gpu_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cols", [(1, 4), (17, 60), (16385, 64), (501, 68), (4099, 128), (301, 132), (39999, 132), (40003, 256),
                                       (5999, 260), (6001, 384), (6007, 512), (4095, 516), (4097, 516), (4101, 1024)])
def test_short_rows(aq, rows, cols):
    print(f"[quantize rows] {rows}x{cols}", flush=True)
    rng = np.random.default_rng(rows + cols)
    w = (rng.standard_normal((rows, cols)) * 0.05).astype(np.float32)
    w[rows // 2] = 0.0
    w[rows - 1] *= np.float32(1e-30)
    codes = torch.zeros(rows * cols, dtype=torch.uint8, device=U.DEV)
    scale = torch.zeros(rows, device=U.DEV)
    zp = torch.full((rows,), 7, dtype=torch.int32, device=U.DEV)
    ws = torch.zeros(4096, dtype=torch.int32, device=U.DEV)
    aq.quantize_tensor(U.to_dev(w), rows, cols, "channel_sym_s8", 255, codes, scale, zp, ws)
    c = codes.cpu().numpy().view(np.int8).reshape(rows, cols)
    amax = np.abs(w).max(axis=1)
    s = np.where(amax == 0, np.float32(1), amax / np.float32(127)).astype(np.float32)
    assert np.array_equal(scale.cpu().numpy(), s) and not zp.cpu().numpy().any()
    assert np.array_equal(c, np.clip(np.rint((w / s[:, None]).astype(np.float32)), -127, 127).astype(np.int8))
    assert int(ws[2]) == 0
    w[rows // 3, cols - 1] = np.nan
    aq.quantize_tensor(U.to_dev(w), rows, cols, "channel_sym_s8", 255, codes, scale, zp, ws)
    assert int(ws[2]) == 1
