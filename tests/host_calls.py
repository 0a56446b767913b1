"""libquan.so on the fake HIP runtime of fake_hip.cpp: calls of the C ABI whose
host side alone runs.  For processes that have loaded no HIP runtime (see
in_child); addresses of tensors are made up and never read."""
import ctypes
import multiprocessing
import os
import subprocess
from collections import namedtuple

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2509_05512_amd", "libquan.so")
F32, BF16 = 0, 1

Event = namedtuple("Event", "what tag stream name ptr bytes in_capture")
_vp, _i, _f = ctypes.c_void_p, ctypes.c_int32, ctypes.c_float


def build(folder):
    so = os.path.join(str(folder), "libfakehip.so")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                           "-I/opt/rocm/include", "-o", so, os.path.join(HERE, "fake_hip.cpp")])
    return so


def in_child(fn, so, *args):
    """fn(Calls, *args) in a process of its own, where the fake runtime is the
    first HIP runtime loaded."""
    with multiprocessing.get_context("spawn").Pool(1) as pool:
        return pool.apply(_run, (fn, so, args))


def _run(fn, so, args):
    return fn(Calls(so), *args)


class Calls:
    def __init__(self, so):
        self.fake = ctypes.CDLL(so, mode=ctypes.RTLD_GLOBAL)
        self.fake.fake_event.restype = ctypes.c_char
        self.fake.fake_capture.argtypes = [_vp, ctypes.c_int]
        self.fake.fake_limit.argtypes = [ctypes.c_size_t]
        self.lib = ctypes.CDLL(LIB)
        self.lib.quan_last_error.restype = ctypes.c_char_p
        self.next = 0x100000000000

    def at(self, nbytes=1 << 32):
        """A made-up device address with room behind it."""
        self.next += (nbytes + (1 << 20)) // (1 << 20) * (1 << 20)
        return _vp(self.next - (nbytes + (1 << 20)) // (1 << 20) * (1 << 20))

    def events(self):
        out = []
        for i in range(self.fake.fake_events()):
            tag, cap, nb = ctypes.c_int(), ctypes.c_int(), ctypes.c_size_t()
            stream, ptr, name = _vp(), _vp(), ctypes.c_char_p()
            what = self.fake.fake_event(i, ctypes.byref(tag), ctypes.byref(stream), ctypes.byref(name),
                                        ctypes.byref(ptr), ctypes.byref(nb), ctypes.byref(cap))
            out.append(Event(what.decode(), tag.value, stream.value, name.value.decode(), ptr.value, nb.value, cap.value))
        return out

    def clear(self):
        self.fake.fake_clear()

    def _ok(self, rc):
        if rc != 0:
            raise RuntimeError(f"{rc}: {self.lib.quan_last_error().decode()}")

    def _sizes(self, n, c_in, h, w, c_out, k, dtype, stream):
        return [_i(v) for v in (n, c_in, h, w, c_out, k, k, dtype)] + [_vp(stream)]

    @staticmethod
    def _geo(stride, pad, dilation=1):
        return [_i(v) for v in (stride, stride, pad, pad, dilation, dilation)]

    # shape: (n, c_in, h, w, c_out, k, stride, pad)
    def forward_packed(self, shape, dtype=BF16, stream=0, sep=False):
        n, c, h, w, o, k, s, p = shape
        fn = self.lib.quan_qconv2d_separable_forward_packed if sep else self.lib.quan_qconv2d_forward_packed
        self._ok(fn(self.at(), self.at(), None, *self._geo(s, p), self.at(),
                    *self._sizes(n, c, h, w, o, k, dtype, stream)))

    def forward(self, shape, dtype=BF16, stream=0):
        n, c, h, w, o, k, s, p = shape
        self._ok(self.lib.quan_qconv2d_forward(self.at(), *[self.at() for _ in range(4)], None, *self._geo(s, p),
                                               self.at(), *self._sizes(n, c, h, w, o, k, dtype, stream)))

    def inference(self, shape, dtype=BF16, stream=0):
        n, c, h, w, o, k, s, p = shape
        self._ok(self.lib.quan_qconv2d_iqbn_inference(
            self.at(), self.at(), None, *self._geo(s, p), *[self.at() for _ in range(4)], _f(1e-5), _i(0), self.at(),
            *self._sizes(n, c, h, w, o, k, dtype, stream)))

    def iqbn_layer(self, shape, dtype=BF16, stream=0, stats=0):
        n, c, h, w, o, k, s, p = shape
        self._ok(self.lib.quan_qconv2d_iqbn_forward(
            self.at(), self.at(), None, *self._geo(s, p), self.at(), self.at(), _f(1e-5), _i(0), _i(stats), self.at(),
            self.at(), self.at(), *self._sizes(n, c, h, w, o, k, dtype, stream)))

    def backward_data(self, shape, dtype=BF16, stream=0):
        n, c, h, w, o, k, s, p = shape
        self._ok(self.lib.quan_qconv2d_backward_data(self.at(), *[self.at() for _ in range(4)], *self._geo(s, p),
                                                     self.at(), *self._sizes(n, c, h, w, o, k, dtype, stream)))

    def backward_weight(self, shape, dtype=BF16, stream=0):
        n, c, h, w, o, k, s, p = shape
        self._ok(self.lib.quan_qconv2d_backward_weight(
            self.at(), self.at(), *self._geo(s, p), *[self.at() for _ in range(5)],
            *self._sizes(n, c, h, w, o, k, dtype, stream)))

    def stem(self, n, h, w, c_out, k, stride, dtype=BF16, stream=0):
        self._ok(self.lib.quan_qconv2d_poincare_forward(
            self.at(), self.at(), None, *self._geo(stride, k // 2), self.at(),
            *[_i(v) for v in (n, h, w, c_out, k, k, dtype)], _vp(stream)))

    def iqbn(self, n, c, h, w, dtype=BF16, stream=0):
        self._ok(self.lib.quan_iqbn_forward(self.at(), self.at(), self.at(), _f(1e-5), self.at(), self.at(), self.at(),
                                            *[_i(v) for v in (n, c, h, w, dtype)], _vp(stream)))

    def iqbn_backward(self, n, c, h, w, dtype=BF16, stream=0, relu=True):
        self._ok(self.lib.quan_iqbn_backward(
            self.at(), self.at(), self.at() if relu else None, self.at(), self.at(), self.at(), _f(1e-5), self.at(),
            self.at(), self.at(), *[_i(v) for v in (n, c, h, w, dtype)], _vp(stream)))
