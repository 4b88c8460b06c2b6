"""The erfcx coefficient table of the device's U-sampler and acceptance scan
(Weideman's rational approximation, erfcx_table.hpp): it is what its
generator writes, and evaluated in the device's form it reproduces
scipy.special.erfcx to the stated 1e-15 relative error on y >= 0."""
import pathlib
import re
import subprocess
import sys

import numpy as np
from scipy.special import erfcx

CSRC = pathlib.Path(__file__).resolve().parents[1] / "paper_2606_13426_amd" / "csrc"


def _table():
    s = (CSRC / "erfcx_table.hpp").read_text()
    L = float(re.search(r"kWeidemanL = ([^;]+);", s).group(1))
    a = [float(x) for x in re.findall(r"^\s+([-0-9.e+]+),$", s, re.M)]
    n = int(re.search(r"kWeidemanN = (\d+);", s).group(1))
    assert len(a) == n
    return L, np.array(a)


def test_table_matches_generator():
    out = subprocess.run([sys.executable, str(CSRC / "gen_erfcx_table.py")], capture_output=True,
                         text=True, check=True).stdout
    assert out == (CSRC / "erfcx_table.hpp").read_text()


def test_table_reproduces_erfcx():
    L, a = _table()
    y = np.concatenate([np.linspace(0.0, 12.0, 48001), np.logspace(-12, 19, 6000), [0.0, 1e300]])
    inv = 1.0 / (L + y)
    z = (L - y) * inv
    # four chains in z^4, each step a fused multiply-add (the long double holds the
    # product of two doubles to 11 more bits), joined as the device joins them
    fma = lambda u, v, w: (u.astype(np.longdouble) * v + w).astype(np.float64)  # noqa: E731
    z2 = z * z
    z4 = z2 * z2
    q = [np.full_like(y, a[j]) for j in range(4)]
    for n in range(4, len(a)):
        q[n % 4] = fma(q[n % 4], z4, a[n])
    p = fma(fma(q[0], z, q[1]), z2, fma(q[2], z, q[3]))
    got = fma(2.0 * p, inv, 1.0 / np.sqrt(np.pi)) * inv
    ref = erfcx(y)
    assert np.all(np.abs(got - ref) <= 1e-15 * ref)
