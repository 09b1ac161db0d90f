"""The plain sampler's polynomials (csrc/cs_icdf_table.h) on the CPU: the tail
series and the small-x total against their definitions, and the header against
its generator (the FP32 starting values, a least-squares fit, to 1e-4 of
their largest coefficient)."""
import os
import re
import subprocess
import sys

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2206_02937_amd", "csrc")


def _array(text, name):
    m = re.search(re.escape(name) + r"(\[\d+\])+ = \{(.*?)\};", text, re.S)
    return np.array([float(v) for v in re.findall(r"[-+]?\d\.\d+e[-+]\d+", m.group(2))])


def _header():
    return open(os.path.join(CSRC, "cs_icdf_table.h")).read()


def test_tail_polynomial_is_the_series():
    c = _array(_header(), "kTailPoly")
    s = np.linspace(0.0, 0.25, 2001)
    k = np.arange(60)
    series = np.sum(2.0 * s[:, None] ** k / (2.0 * k + 3.0), axis=1)
    e = np.zeros_like(s)
    for a in c[::-1]:
        e = e * s + a
    assert np.max(np.abs(e - series) / series) <= 6e-16  # rounding of the two sums


def test_small_x_total(orc):
    c = _array(_header(), "kSmallZ")
    x = np.concatenate([[0.0, 1e-300], 10.0 ** np.linspace(-12, np.log10(2.0 ** -8), 300)])
    got = np.polyval(c[::-1], x)
    ref = np.array([8.0 / 3.0 * orc.sigma_ratio(float(v)) for v in x])
    assert np.max(np.abs(got - ref) / ref) <= 1e-14  # the oracle's own bound on s(x)


def test_header_is_what_the_generator_writes(tmp_path):
    code = open(os.path.join(CSRC, "gen_icdf_table.py")).read()
    code = code.replace('OUT = os.path.join(HERE, "cs_icdf_table.h")', f'OUT = {str(tmp_path / "t.h")!r}')
    script = tmp_path / "gen.py"
    script.write_text(code)
    subprocess.run([sys.executable, str(script)], check=True, capture_output=True)
    new, old = (tmp_path / "t.h").read_text(), _header()
    for name in ("kTailPoly", "kSmallZ"):
        assert np.array_equal(_array(new, name), _array(old, name)), name
    for name in ("kStart", "kStartA", "kStartB", "kStartTail"):
        a, b = _array(new, name), _array(old, name)
        assert np.max(np.abs(a - b)) <= 1e-4 * np.max(np.abs(b)), name
