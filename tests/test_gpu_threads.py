"""Two host threads on one stream, whose layers hand data from one launch to
the next through buffers of the stream (a padded input, partial tiles, packed
kernels): every result has the bits that one thread gets."""
import threading

import pytest
import torch

from paper_2509_05512_amd import quan
from parity import say

pytestmark = pytest.mark.gpu

# (n, c_in, h, w, c_out): 3x3, bf16; padded (12, 20, 3 channels), split, whole
LAYERS = [(8, 12, 20, 20, 20), (1, 128, 7, 7, 64), (8, 20, 33, 31, 16), (1, 256, 14, 14, 128), (2, 3, 40, 41, 32),
          (4, 32, 28, 28, 32)]


def _layer(i, shape):
    n, c, h, w, o = shape
    g = torch.Generator().manual_seed(i)
    x = quan.to_device_layout(torch.randn(n, 4, c, h, w, generator=g).to(torch.bfloat16).cuda())
    ws = [(torch.randn(o, c, 3, 3, generator=g) * 0.1).to(torch.bfloat16).cuda() for _ in range(4)]
    return x, ws, quan.quan_qconv2d_pack_weights(*ws)


@pytest.mark.parametrize("packed", [True, False], ids=["packed", "unpacked"])
def test_two_threads_on_one_stream(packed):
    say(f"two threads on one stream, packed={packed}")
    layers = [_layer(i, s) for i, s in enumerate(LAYERS)]

    def call(layer):
        x, ws, p = layer
        if packed:
            return quan.quan_qconv2d_forward_packed(x, p, tuple(ws[0].shape), pad=1)
        return quan.quan_qconv2d_forward(x, *ws, pad=1)

    want = [call(layer) for layer in layers]
    torch.cuda.synchronize()
    got, failed = {0: [], 1: []}, []

    def run(tag):
        try:
            for _ in range(20):
                for i in (range(len(layers)) if tag == 0 else reversed(range(len(layers)))):
                    got[tag].append((i, call(layers[i])))
        except Exception as e:  # noqa: BLE001
            failed.append(repr(e))

    threads = [threading.Thread(target=run, args=(t,)) for t in (0, 1)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not failed, failed
    for tag in got:
        assert len(got[tag]) == 20 * len(layers)
        for i, y in got[tag]:
            assert torch.equal(y, want[i]), f"thread {tag}, layer {LAYERS[i]}"


def test_call_beside_a_capture():
    """Another thread's calls that allocate and outgrow the buffers of their own
    stream leave a capture in progress alone."""
    say("calls beside another thread's capture")
    held, small, large, whole = [_layer(10 + i, s) for i, s in enumerate(
        [(4, 32, 28, 28, 32), (2, 12, 20, 20, 20), (8, 12, 40, 40, 20), (64, 32, 32, 32, 64)])]

    def call(layer, out):
        return quan.quan_qconv2d_forward_packed(layer[0], layer[2], tuple(layer[1][0].shape), pad=1, out=out)

    outs = [torch.empty_like(quan.quan_qconv2d_forward_packed(x, p, tuple(ws[0].shape), pad=1))
            for x, ws, p in (held, small, large, whole)]
    want = [call(layer, None) for layer in (held, small, large)]
    mine, other = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for st in (mine, other):
        with torch.cuda.stream(st):
            call(whole, outs[3])
    torch.cuda.synchronize()
    failed = []

    def run():
        try:
            with torch.cuda.stream(other):
                call(small, outs[1])
                call(large, outs[2])
        except Exception as e:  # noqa: BLE001
            failed.append(repr(e))

    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=mine):
        call(held, outs[0])
        t = threading.Thread(target=run)
        t.start()
        t.join()
    torch.cuda.synchronize()
    assert not failed, failed
    for _ in range(3):
        outs[0].fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(outs, want))
