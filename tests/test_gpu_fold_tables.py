"""Inference layers whose launch forms the folded map itself, one table per
work-group: channel counts around 256 columns (one per compute thread), several
channel tiles, direct and deferred stores, both types, with and without bias
and ReLU; a layer too wide for tables on that many work-groups; two streams at
once.  Against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_05512_amd import quan
from parity import assert_close, f64, say

pytestmark = pytest.mark.gpu

DT = {"fp32": torch.float32, "bf16": torch.bfloat16}

# (N, Cin, Cout, H, W, k, stride)
CASES = [("bf16", (2, 8, c, 24, 25, 3, 1)) for c in (5, 12, 16, 63, 64, 65, 72, 136)]
CASES += [("fp32", (2, 4, c, 16, 15, 3, 1)) for c in (3, 16, 63, 65)]
CASES += [("bf16", (16, 32, 64, 40, 40, 3, 2)), ("bf16", (1, 8, 2100, 33, 34, 1, 1))]


def _make(dtype, case, seed):
    N, Cin, Cout, H, W, k, s = case
    rng = np.random.default_rng(seed)
    dt = DT[dtype]
    x = torch.from_numpy(rng.standard_normal((N, 4, Cin, H, W), dtype=np.float32)).to(dt)
    w = torch.from_numpy((rng.standard_normal((4, Cout, Cin, k, k)) / np.sqrt(4 * Cin * k * k)).astype(np.float32)).to(dt)
    b = torch.from_numpy((rng.standard_normal((4, Cout)) * 0.3).astype(np.float32)).to(dt)
    f = [torch.from_numpy(v.astype(np.float32)) for v in
         (rng.standard_normal((4, Cout)) * 0.5, rng.uniform(0.5, 2.0, (4, Cout)), rng.uniform(0.5, 1.5, (4, Cout)),
          rng.standard_normal((4, Cout)) * 0.3)]
    return x, w, b, f


def _serve(x, w, b, f, k, s, relu):
    ws = [w[q].contiguous().cuda() for q in range(4)]
    return quan.quan_qconv2d_iqbn_inference(quan.to_device_layout(x.cuda()), quan.quan_qconv2d_pack_weights(*ws),
                                            tuple(ws[0].shape), *[t.cuda() for t in f],
                                            bias=b.cuda() if b is not None else None, stride=s, pad=k // 2, relu=relu)


def _ref(x, w, b, f, k, s, relu):
    y = oracle.qconv2d(f64(x), f64(w), f64(b) if b is not None else None, s, k // 2, 1)
    return oracle.iqbn_inference(y, *[f64(t) for t in f], 1e-5, relu)


@pytest.mark.parametrize("relu", [False, True], ids=["plain", "relu"])
@pytest.mark.parametrize("dtype,case", CASES, ids=[f"{t}-{c}" for t, c in CASES])
def test_fold_tables(dtype, case, relu):
    say(f"fold tables {dtype} {case} relu={relu}")
    x, w, b, f = _make(dtype, case, sum(case))
    k, s = case[5:]
    if not relu:
        b = None
    z = _serve(x, w, b, f, k, s, relu)
    torch.cuda.synchronize()
    assert_close(f64(z), _ref(x, w, b, f, k, s, relu), DT[dtype], f"{case}")


def test_fold_tables_two_streams():
    say("fold tables, two streams")
    cases = [(4, 16, 64, 60, 60, 3, 1), (4, 16, 40, 60, 60, 3, 1)]
    data = [_make("bf16", c, 11 + i) for i, c in enumerate(cases)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    outs = []
    torch.cuda.synchronize()
    for (x, w, b, f), st in zip(data, streams):
        with torch.cuda.stream(st):
            outs.append([_serve(x, w, b, f, 3, 1, True) for _ in range(3)])
    torch.cuda.synchronize()
    for (x, w, b, f), out in zip(data, outs):
        ref = _ref(x, w, b, f, 3, 1, True)
        for z in out:
            assert_close(f64(z), ref, torch.bfloat16, "two streams")
