"""cl_quantize_pack and cl_dequantize against the oracle: bit-exact codes,
scales, zeros and dequantized values (Section 5.1 backbone quantizer, RTN
reading of GPTQ without calibration data)."""

import numpy as np
import pytest
import torch

from oracle import quant
from paper_2605_05819_amd import cl, workloads as wl
from tests.helpers import dev_u32, dev_f16, host_u16, host_u32

pytestmark = pytest.mark.gpu


def _adversarial(bits, G, rows):
    """Rows that stress the rounding rules: exact ties, constant and zero
    groups, one-sided groups, clamped maxima, tiny and huge magnitudes."""
    g = np.random.default_rng(1234 + bits)
    qmax = (1 << bits) - 1
    d_in = 4 * G
    W = (0.02 * g.standard_normal((rows, d_in))).astype(np.float64)
    step = 2.0 ** -8
    # exact half-steps on a power-of-two grid -> ties to even
    W[0, :G] = step * (np.resize(np.arange(-3, qmax - 2) + 0.5, G))
    W[0, 0], W[0, 1] = -3 * step, (qmax - 3) * step
    W[1, :G] = 0.0                                  # all-zero group
    W[1, G:2 * G] = 0.37                            # constant positive group
    W[1, 2 * G:3 * G] = -0.01                       # constant negative group
    W[2, :G] = np.abs(W[2, :G])                     # one-sided
    W[2, G:2 * G] = -np.abs(W[2, G:2 * G])
    W[3, :G] *= 1e-6                                # subnormal-range scale
    W[3, G:2 * G] *= 1e-9                           # scale rounds to 0 -> held at 2^-24
    W[4, :G] *= 1e5                                 # huge values: scale beyond fp16 -> 65504
    return W.astype(np.float32)


@pytest.mark.parametrize("bits,G", [(4, 128), (2, 64), (4, 32), (2, 128), (3, 128), (3, 32)])
def test_quantize_pack_bit_exact(bits, G):
    rows = 37                                       # ragged: not a multiple of anything
    W = np.concatenate([_adversarial(bits, G, 8),
                        wl.weight((rows - 8, 4 * G), 0, 0, bits, G)], axis=0)
    w = cl.quantize_pack(torch.from_numpy(W).cuda(), bits, G)
    torch.cuda.synchronize()
    Q, s, z = quant.quantize_pack(W, bits, G)
    np.testing.assert_array_equal(host_u32(w.q), Q)
    np.testing.assert_array_equal(host_u16(w.scales), s.view(np.uint16))
    np.testing.assert_array_equal(host_u16(w.zeros), z.view(np.uint16))


def test_quantize_pack_llama_gate_rows_bit_exact():
    """Full 14336 x 4096 gate matrix quantized on the GPU; rows sampled across
    the whole matrix (quantization is row-independent) checked bit-exactly."""
    W = wl.weight((14336, 4096), 1, 0, 4)
    w = cl.quantize_pack(torch.from_numpy(W).cuda(), 4, 128)
    torch.cuda.synchronize()
    rows = np.r_[0:3, np.random.default_rng(0).choice(14336, 60, replace=False), 14333:14336]
    Q, s, z = quant.quantize_pack(W[rows], 4, 128)
    np.testing.assert_array_equal(host_u32(w.q)[rows], Q)
    np.testing.assert_array_equal(host_u16(w.scales)[rows], s.view(np.uint16))
    np.testing.assert_array_equal(host_u16(w.zeros)[rows], z.view(np.uint16))


@pytest.mark.parametrize("bits,G", [(4, 128), (2, 64), (3, 128), (3, 32)])
def test_dequantize_exact(bits, G):
    W = wl.weight((50, 512), 0, 3, bits)
    Q, s, z = quant.quantize_pack(W, bits, G)
    w = cl.QWeight(dev_u32(Q), dev_f16(s), dev_f16(z), 50, 512, bits, G)
    got = cl.dequantize(w).cpu().numpy().astype(np.float64)
    np.testing.assert_array_equal(got, quant.dequant_packed(Q, s, z, bits, G, 512))


def test_quantize_pack_3bit_llama_rows_bit_exact():
    """3-bit codes (32 in 3 words, two of them straddling words) of a full
    14336 x 4096 matrix quantized on the GPU, sampled rows bit-exact."""
    W = wl.weight((14336, 4096), 7, 0, 4)
    w = cl.quantize_pack(torch.from_numpy(W).cuda(), 3, 128)
    torch.cuda.synchronize()
    assert tuple(w.q.shape) == (14336, 384)
    rows = np.r_[0:2, np.random.default_rng(3).choice(14336, 40, replace=False), 14334:14336]
    Q, s, z = quant.quantize_pack(W[rows], 3, 128)
    np.testing.assert_array_equal(host_u32(w.q)[rows], Q)
    np.testing.assert_array_equal(host_u16(w.scales)[rows], s.view(np.uint16))
    np.testing.assert_array_equal(host_u16(w.zeros)[rows], z.view(np.uint16))


@pytest.mark.parametrize("bits,G,rows,offset", [
    (4, 32, 1, 0), (4, 96, 5, 0), (4, 256, 37, 1), (4, 512, 37, 0), (4, 1024, 9, 1),   # lanes of a group: 4 .. 64, a wave
    (3, 32, 3, 1), (3, 96, 4, 0), (3, 512, 5, 0), (3, 640, 2, 1),
    (2, 64, 1, 1), (2, 192, 7, 0), (2, 512, 3, 0), (2, 1088, 2, 1),
])
def test_every_group_width_and_alignment_bit_exact(bits, G, rows, offset):
    """Group sizes on both kernels, odd row counts, a weight and an output
    that start 4 bytes past a 16-byte boundary, values next to every tie of
    the grid (the fp32 decision falls back to fp64 there), infinities'
    neighbourhood and an empty-range group."""
    d_in = 4 * G if bits != 3 else 128 * G // np.gcd(128, G)
    g = np.random.default_rng(G + bits)
    W = (0.02 * g.standard_normal((rows, d_in))).astype(np.float32)
    qmax = (1 << bits) - 1
    step = np.float32(0.0078125)
    ties = ((np.arange(G) % qmax) - 1.5).astype(np.float32) * step
    W[0, :G] = np.where(np.arange(G) % 3 == 0, ties, np.nextafter(ties, np.float32(np.inf) * (-1.0) ** np.arange(G)))
    W[0, 0], W[0, 1] = -2 * step, (qmax - 2) * step
    W[0, G:2 * G] = 3.0e38 * np.sign(W[0, G:2 * G])
    W[-1, -G:] = 0.0
    host = torch.from_numpy(W)
    buf = torch.empty(W.size + offset, dtype=torch.float32, device="cuda")
    Wd = buf[offset:].view(rows, d_in)
    Wd.copy_(host)
    w = cl.quantize_pack(Wd, bits, G)
    Q, s, z = quant.quantize_pack(W, bits, G)
    np.testing.assert_array_equal(host_u32(w.q), Q)
    np.testing.assert_array_equal(host_u16(w.scales), s.view(np.uint16))
    np.testing.assert_array_equal(host_u16(w.zeros), z.view(np.uint16))
    import ctypes
    out = torch.full((W.size + 2,), 7.0, dtype=torch.float32, device="cuda")
    qc = w.c()
    at = out[offset:]
    assert cl.lib().cl_dequantize(ctypes.byref(qc), ctypes.c_void_p(at.data_ptr()), None) == 0
    torch.cuda.synchronize()
    ref = quant.dequant_packed(Q, s, z, bits, G, d_in).astype(np.float32).reshape(-1)
    np.testing.assert_array_equal(at[:W.size].cpu().numpy(), ref)
    assert (out[offset + W.size:] == 7.0).all()
