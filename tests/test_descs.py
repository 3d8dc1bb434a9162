"""The frame records handed to the library, against the specs they were built from, for every
form of gains and shifts a spec may carry; records of one spec repeated; no aliasing of the
gains."""
import numpy as np
import pytest

import paper_2604_02266_amd as otfs


class Spec:
    def __init__(self, h, tau, nu, qam=4):
        self.M, self.N, self.lam, self.qam = 16, 8, 0.25, qam
        self.h, self.tau, self.nu = h, tau, nu


G = np.array([0.5 + 0.25j, -0.125 - 1j, 0.75j])
FORMS = {
    "complex128": (G, np.arange(3), np.arange(3) - 1),
    "complex64": (G.astype(np.complex64), np.arange(3, dtype=np.int32), np.arange(3, dtype=np.int16)),
    "lists": (list(G), [2, 0, 1], [-1, 0, 1]),
    "strided": (np.repeat(G, 2)[::2], np.arange(6)[::2], np.arange(6, dtype=np.int32)[::-2]),
    "real": (G.real, np.arange(3.0), np.arange(3)),
    "column": (G[:, None], np.arange(3), np.arange(3)),
}


def check(d, f):
    h = np.asarray(f.h).reshape(-1).astype(np.complex64)
    assert (d.M, d.N, d.P, d.noise_var, d.qam) == (16, 8, 3, 0.25, f.qam or 0)
    assert [d.h[i] for i in range(6)] == [v for z in h for v in (z.real, z.imag)]
    assert [d.delay[i] for i in range(3)] == [int(v) for v in f.tau]
    assert [d.doppler[i] for i in range(3)] == [int(v) for v in f.nu]


@pytest.mark.parametrize("form", sorted(FORMS))
def test_records_hold_the_specs(form):
    a, b = Spec(*FORMS[form]), Spec(*FORMS["complex128"], qam=None)
    frames = [a, a, b, a]
    d = otfs._Descs(frames)
    assert len(d.arr) == 4
    for i, f in enumerate(frames):
        check(d.arr[i], f)


def test_records_of_no_frames_and_gains_copied():
    assert len(otfs._Descs([]).arr) == 1
    h = G.astype(np.complex64)
    d = otfs._Descs([Spec(h, [0, 1, 2], [0, 0, 0])])
    h[0] = 9
    assert d.arr[0].h[0] == 0.5


def test_values_beyond_the_fields_as_ctypes_stores_them():
    f = Spec(G, [0, 1, 2], [0, 0, 0], qam=2 ** 33 + 4)
    f.M, f.N, f.lam = 2 ** 31, np.int64(2 ** 32 + 8), 1e39
    d = otfs._Descs([f]).arr[0]
    assert (d.M, d.N, d.qam, d.noise_var) == (-2 ** 31, 8, 4, float("inf"))
