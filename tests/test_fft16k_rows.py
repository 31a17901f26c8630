"""CPU model of the 32 x 32 x 16 form of the 16384-point FFT in
csrc/tfx_fft16k.h: 512 threads of 32 values, one exchange through rows of an
LDS plane and one inside a wave's own rows.  The passes run in FP64 with the
kernel's address maps written out again here; checked are the maps (in range,
one-to-one, read back by the writing wave where no barrier stands between),
the composition against numpy's FFT, the inverse, the stored order of the
spectrum, and that no access has a bank conflict."""
import numpy as np

NB, WG, R, ROW = 16384, 512, 32, 528
T = np.arange(WG)
K = np.arange(R)
C = T & 15


def cols():  # [t, k]
    return T[:, None] + ROW * K[None, :]


def rows():
    return (ROW * (T >> 4) + C)[:, None] + 16 * K[None, :]


def rot():
    return (ROW * (T >> 4))[:, None] + 4 * (((C >> 2)[:, None] + (K >> 2)[None, :]) & 3) + (C & 3)[:, None] \
        + 16 * K[None, :]


def grp():  # [t, 16 h + 4 g + i]
    out = np.empty((WG, R), int)
    for h in range(2):
        for g in range(4):
            base = ROW * (T >> 4) + 16 * C + 4 * ((g + (C >> 2)) & 3) + 256 * h
            out[:, 16 * h + 4 * g:16 * h + 4 * g + 4] = base[:, None] + np.arange(4)
    return out


def spec_at(k):
    t = (k & 31) * 16 + ((k >> 5) & 15)
    j = 16 * ((k >> 9) & 1) + (k >> 10)
    return ((j >> 1) * WG + t) * 2 + (j & 1)


def exchange(v, w, r):
    P = np.full(R * ROW, np.nan + 0j)
    P[w] = v
    return P[r]


def forward(z):
    w = lambda m: np.exp(-2j * np.pi * (m % NB) / NB)  # noqa: E731
    v = np.fft.fft(z.reshape(R, WG).T, axis=1)
    v = exchange(v, cols(), rows())                            # thread (k1, c) over b
    v = np.fft.fft(v * w(16 * (T >> 4)[:, None] * K), axis=1)
    v = exchange(v, rot(), grp())                              # thread (k1, k2 mod 16) over c, two halves
    out = []
    for h in range(2):
        kappa = (T >> 4) + 32 * C + 512 * h
        out.append(np.fft.fft(v[:, 16 * h:16 * h + 16] * w(kappa[:, None] * np.arange(16)), axis=1))
    return np.concatenate(out, axis=1)


def inverse(v):
    w = lambda m: np.exp(2j * np.pi * (m % NB) / NB)  # noqa: E731
    halves = []
    for h in range(2):
        kappa = (T >> 4) + 32 * C + 512 * h
        halves.append(16 * np.fft.ifft(v[:, 16 * h:16 * h + 16], axis=1) * w(kappa[:, None] * np.arange(16)))
    v = exchange(np.concatenate(halves, axis=1), grp(), rot())
    v = exchange(32 * np.fft.ifft(v, axis=1), rows(), cols())  # thread t = 16 b + c over k1
    return (32 * np.fft.ifft(v * w(16 * (T >> 4)[:, None] * K), axis=1)).T.reshape(-1)


def test_butterflies_with_turned_inputs():
    """The four-point butterfly whose inputs carry twiddles as tan and cos, with
    the table's stand-in for a cosine of zero."""
    g = np.random.default_rng(2)
    for _ in range(200):
        phi = 2 * np.pi * g.integers(0, 1024, 3) / 1024
        x = g.standard_normal(4) + 1j * g.standard_normal(4)
        c = np.cos(phi)
        c = np.where(np.abs(c) < 2.0 ** -28, 2.0 ** -28, c)
        t = np.sin(phi) / c
        y = x[1:] * (1 - 1j * t)                               # e^{-i phi} / cos phi
        a, b = x[0] + c[1] * y[1], x[0] - c[1] * y[1]
        p, m = y[0] + c[2] / c[0] * y[2], y[0] - c[2] / c[0] * y[2]
        got = np.array([a + c[0] * p, b - 1j * c[0] * m, a - c[0] * p, b + 1j * c[0] * m])
        ref = np.fft.fft(x * np.exp(-1j * np.concatenate([[0.0], phi])))
        assert np.max(np.abs(got - ref)) < 1e-7


def test_maps_are_one_to_one_and_in_range():
    sets = [np.sort(m().ravel()) for m in (cols, rows, rot, grp)]
    for s in sets:
        assert s[0] >= 0 and s[-1] < R * ROW and np.unique(s).size == NB
        assert np.array_equal(s, sets[0])


def test_rows_are_private_to_a_wave():
    wave = T >> 6
    for m in (rows, rot, grp):
        assert np.array_equal((m() // ROW) >> 2, np.broadcast_to(wave[:, None], (WG, R)))


def test_transform_and_inverse():
    g = np.random.default_rng(1)
    z = g.standard_normal(NB) + 1j * g.standard_normal(NB)
    v = forward(z)
    Z = np.fft.fft(z)
    k = np.arange(NB)
    pos = spec_at(k)
    assert np.array_equal(np.sort(pos), k)
    stored = np.empty(NB, complex)
    stored[pos] = Z                                            # [j / 2][t][j % 2]
    got = v.reshape(WG, R // 2, 2).transpose(1, 0, 2).ravel()
    assert np.max(np.abs(got - stored)) < 1e-10
    assert np.max(np.abs(inverse(v) - NB * z)) < 1e-9


def test_no_bank_conflicts():
    for m in (cols, rows, rot):
        a = m() % 64
        for w in range(0, WG, 64):
            for k in range(R):
                assert np.unique(a[w:w + 64, k]).size == 64
    b = grp()[:, ::4] % 64                                     # 16-byte accesses, 16 lanes a phase
    for w in range(0, WG, 16):
        for k in range(R // 4):
            banks = (b[w:w + 16, k][:, None] + np.arange(4)).ravel()
            assert np.unique(banks).size == 64
