"""IQBN forward and gradient at the edges of the one-launch form of small
tensors (its work-group holds 1024 rows of 64-byte column groups, 128 rows
where the columns move one by one), one row past them, and at sizes where the
three-launch form splits into few rows per thread; against the oracle, with
the tolerances of parity.py.  The gradient's ReLU form keeps the sign bits of
the saved output between its passes."""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_05512_amd import quan
from parity import assert_close, f64, say

pytestmark = pytest.mark.gpu

DT = {"fp32": torch.float32, "bf16": torch.bfloat16}

# (N, C, H, W)
SHAPES = [
    (1, 1, 1, 1), (1, 2, 1, 3), (1, 16, 1, 127), (1, 16, 1, 128), (1, 16, 3, 43),
    (1, 24, 31, 33),          # 1023 rows
    (1, 24, 32, 32),          # 1024: the last small one
    (1, 24, 25, 41),          # 1025
    (2, 10, 5, 7), (1, 3, 8, 16), (1, 3, 3, 43), (3, 5, 11, 13),
    (1, 300, 7, 7),           # many column groups, the last one short in fp32
    (5, 20, 25, 27),          # three launches, a block's rows not a whole round
    (1, 256, 32, 32), (1, 257, 32, 32),  # fp32: 4 MiB, and the first forward of the merged form
    (1, 231, 25, 41), (3, 55, 31, 30),   # bf16 rows read element by element, three launches
]


@pytest.mark.parametrize("relu", [False, True], ids=["plain", "relu"])
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=[str(s) for s in SHAPES])
def test_small_tensors(shape, dtype, relu):
    say(f"iqbn small {dtype} {shape} relu={relu}")
    N, C, H, W = shape
    dt = DT[dtype]
    rng = np.random.default_rng(sum(shape) + relu)
    x = torch.from_numpy((rng.standard_normal((N, 4, C, H, W)) * 1.5 + 3.0).astype(np.float32)).to(dt)
    g = torch.from_numpy(rng.uniform(0.5, 1.5, (4, C)).astype(np.float32))
    be = torch.from_numpy((rng.standard_normal((4, C)) * 0.3).astype(np.float32))
    dout = torch.from_numpy(rng.standard_normal((N, 4, C, H, W)).astype(np.float32)).to(dt)
    xg = quan.to_device_layout(x.cuda())
    fwd = quan.quan_iqbn_relu_forward if relu else quan.quan_iqbn_forward
    y, mean, var = fwd(xg, g.cuda(), be.cuda())
    held = xg.clone()
    inplace, _, _ = fwd(held, g.cuda(), be.cuda(), out=held)
    dg_in = quan.to_device_layout(dout.cuda())
    args = (xg, dg_in, mean, var, g.cuda())
    dx, dgamma, dbeta = quan.quan_iqbn_backward(*args, y=y if relu else None)
    over = dg_in.clone()
    dx2, _, _ = quan.quan_iqbn_backward(xg, over, mean, var, g.cuda(), y=y if relu else None, dx=over)
    torch.cuda.synchronize()
    ref, m_ref, v_ref = oracle.iqbn(f64(x), f64(g), f64(be), 1e-5, relu)
    # statistics are fp32 whatever the type of x
    assert_close(f64(mean), m_ref, torch.float32, f"mean {shape}")
    assert_close(f64(var), v_ref, torch.float32, f"var {shape}")
    assert torch.equal(y, inplace) and torch.equal(dx, dx2)
    if N * H * W > 4:  # (var ~ eps on a handful of rows scales rounding up)
        assert_close(f64(y), ref, dt, f"out {shape}")
        mask = (y.cpu().float() > 0).double().numpy() if relu else 1.0
        rdx, rdg, rdb = oracle.iqbn_backward(f64(x), f64(g), f64(be), f64(dout) * mask, 1e-5, False)
        assert_close(f64(dx), rdx, dt, f"dx {shape}")
        # sums of up to 3375 products; bf16 operands are exact in fp32
        assert_close(f64(dgamma), rdg, torch.float32, f"dgamma {shape}")
        assert_close(f64(dbeta), rdb, torch.float32, f"dbeta {shape}")
