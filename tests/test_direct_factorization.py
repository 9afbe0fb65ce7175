"""The direct form's two column passes on the CPU (no GPU): a numpy model with
the kernels' index maps (blocked buffer between the passes, the top-level
factor as w_N^{-v j} w_{16 M1}^{-v r}, the 2^14-point radix-2 step) against
numpy's FFT, for the single kernels' tile width and the batched kernel's."""
import numpy as np
import pytest


def _two_passes(x, l1, l2, lt2):
    """Pass A and pass B of N = 2^l1 2^l2 with 2^lt2 columns per pass-B tile."""
    M1, M2, N = 1 << l1, 1 << l2, 1 << (l1 + l2)
    A = np.fft.fft(x.reshape(M1, M2), axis=0)                     # A[k1, c]
    ws = np.full(N, np.nan, complex)
    k, c = np.meshgrid(np.arange(M1), np.arange(M2), indexing="ij")
    ws[((k >> lt2) << (l2 + lt2)) + (c << lt2) + (k & ((1 << lt2) - 1))] = A
    assert not np.isnan(ws).any()                                 # every item written once
    y = np.empty(N, complex)
    rows, t = np.meshgrid(np.arange(M2), np.arange(1 << lt2), indexing="ij")
    j, r = rows & (M2 // 16 - 1), rows >> (l2 - 4)
    for col0 in range(0, M1, 1 << lt2):
        v = col0 + t
        z = ws[(col0 << l2) + (rows << lt2) + t]
        z = z * np.exp(-2j * np.pi * ((v * j) % N) / N) * np.exp(-2j * np.pi * ((v * r) % (16 * M1)) / (16 * M1))
        y.reshape(M2, M1)[:, col0:col0 + (1 << lt2)] = np.fft.fft(z, axis=0)
    return y


@pytest.mark.parametrize("l1,l2,lt2", [(8, 7, 2), (8, 7, 7), (7, 8, 6), (8, 8, 6), (9, 8, 2), (7, 10, 4), (10, 7, 7),
                                       (10, 10, 4), (11, 10, 2)])
def test_two_passes_are_the_dft(l1, l2, lt2):
    rng = np.random.default_rng(l1 * 16 + l2)
    x = rng.standard_normal(1 << (l1 + l2)) + 1j * rng.standard_normal(1 << (l1 + l2))
    ref = np.fft.fft(x)
    assert np.linalg.norm(_two_passes(x, l1, l2, lt2) - ref) <= 1e-12 * np.linalg.norm(ref)


def test_radix_2_step_of_2_14_points():
    rng = np.random.default_rng(14)
    x = rng.standard_normal(1 << 14) + 1j * rng.standard_normal(1 << 14)
    E, O = np.fft.fft(x[0::2]), np.fft.fft(x[1::2])
    y = np.empty(1 << 14, complex)
    j = np.arange(4096)                                           # = tid + 512 i
    w = np.exp(-2j * np.pi * (j & 511) / (1 << 14)) * np.exp(-2j * np.pi * (4 * (j >> 9)) * 128 / (1 << 14))
    o0, o1 = O[:4096] * w, O[4096:] * w * -1j
    for q, v in enumerate((E[:4096] + o0, E[4096:] + o1, E[:4096] - o0, E[4096:] - o1)):
        y[j + 4096 * q] = v
    ref = np.fft.fft(x)
    assert np.linalg.norm(y - ref) <= 1e-12 * np.linalg.norm(ref)
