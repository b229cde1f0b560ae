"""Error of the transforms against FP64, held to that of separate twiddle products.

`product_form` carries out the engine's Stockham passes with one rounded
twiddle pair per value ahead of radix-4 steps, every operation rounded to the
working type.  A kernel in that arithmetic differs from it only where the
compiler contracts a product into a sum (one rounding less), so its RMS error
may exceed the emulation's by the spread of an RMS over M independent values,
1 / (2 sqrt(M)): 0.1% at M = 2^18.  The bar is five of these.
"""
import numpy as np
import pytest

import oracle
from paper_2605_28451_amd import api, scenes
from tests.gpu_util import announce, download, need_gpu, rand_rows, upload

pytestmark = pytest.mark.gpu

VALUES = 1 << 18
BAR = 1.005
RADICES = {32: (16, 2), 64: (16, 4), 128: (16, 8), 256: (16, 16), 512: (8, 8, 8), 1024: (16, 16, 4),
           2048: (16, 16, 8), 4096: (16, 16, 16), 8192: (16, 16, 16, 2), 16384: (16, 16, 16, 4)}
RADICES1 = {512: (16, 16, 2), 1024: (8, 8, 8, 2)}  # the second radix plan


class Pair:
    """Complex arrays of one floating type; products as the kernels form them."""

    def __init__(self, re, im):
        self.re, self.im = re, im

    def __add__(self, o):
        return Pair(self.re + o.re, self.im + o.im)

    def __sub__(self, o):
        return Pair(self.re - o.re, self.im - o.im)

    def mi(self):  # times -i
        return Pair(self.im, -self.re)

    def scaled(self, k):
        return Pair(self.re * self.re.dtype.type(k), self.im * self.re.dtype.type(k))

    def times(self, wr, wi):
        dt = self.re.dtype
        wr, wi = np.asarray(wr).astype(dt), np.asarray(wi).astype(dt)

        def fma(a, b, c):
            return (a.astype(np.float64) * b.astype(np.float64) + c.astype(np.float64)).astype(dt)
        return Pair(fma(self.re, wr, -(self.im * wi)), fma(self.im, wr, self.re * wi))

    def value(self):
        return self.re.astype(np.float64) + 1j * self.im.astype(np.float64)


def _pair(z, dt):
    return Pair(z.real.astype(dt), z.imag.astype(dt))


def _dft4(a, b, c, d):
    s0, s1, s2, s3 = a + c, a - c, b + d, b - d
    return [s0 + s2, s1 + s3.mi(), s0 - s2, s1 - s3.mi()]


def _turn(a, e, r):  # times W_r^e
    e %= r
    if e == 0:
        return a
    if 4 * e == r:
        return a.mi()
    if 8 * e == r:
        return (a + a.mi()).scaled(np.sqrt(0.5))
    if 8 * e == 3 * r:
        return (a.mi() - a).scaled(np.sqrt(0.5))
    return a.times(np.cos(2 * np.pi * e / r), -np.sin(2 * np.pi * e / r))


def _dft(v):
    r = len(v)
    if r == 2:
        return [v[0] + v[1], v[0] - v[1]]
    if r == 4:
        return _dft4(*v)
    if r == 8:
        e, o = _dft4(*v[0::2]), _dft4(*v[1::2])
        o = [_turn(o[k], k, 8) for k in range(4)]
        return [e[k] + o[k] for k in range(4)] + [e[k] - o[k] for k in range(4)]
    y = [_dft4(*v[n::4]) for n in range(4)]
    out = [None] * 16
    for k in range(4):
        out[k::4] = _dft4(*[_turn(y[n][k], n * k, 16) for n in range(4)])
    return out


def product_form(x, radices, dt):
    """Forward transforms of the rows of complex `x` in the arithmetic `dt`."""
    rows, n = x.shape
    z, ns = _pair(x, dt), 1
    for r in radices:
        v = [Pair(z.re.reshape(rows, r, -1)[:, k], z.im.reshape(rows, r, -1)[:, k]) for k in range(r)]
        if ns > 1:
            m = np.arange(n // r) % ns
            w = np.exp(-2j * np.pi * np.arange(ns * r) / (ns * r))
            v = [v[0]] + [v[k].times(w[m * k].real, w[m * k].imag) for k in range(1, r)]
        v = _dft(v)

        def scatter(part):
            return np.stack([part(a).reshape(rows, -1, ns) for a in v], axis=2).reshape(rows, n)
        z, ns = Pair(scatter(lambda a: a.re), scatter(lambda a: a.im)), ns * r
    return z.value()


def rms(z):
    return float(np.sqrt(np.mean(np.abs(z) ** 2)))


def check(got, ref, emulated, what):
    ratio = rms(got - ref) / rms(emulated - ref)
    print(f"[measure] precision.{what} error {rms(got - ref) / rms(ref):.4e}, {ratio:.4f} of the product form's")
    assert ratio <= BAR


@pytest.mark.parametrize("n", [4096, 8192, 16384])
def test_fp16_forward_error(n):
    need_gpu()
    rows = VALUES // n
    announce(f"fp16 forward error {rows}x{n}")
    x = scenes.quantize(rand_rows(rows, n, n), "fp16")
    got = download(api.FFTPlan(n, rows, "fp16").forward(upload(x, "fp16")), "fp16")
    check(got, oracle.fft(x), product_form(x, RADICES[n], np.float16), f"fp16.n{n}")
