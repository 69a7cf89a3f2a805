"""Host-only rules that decide which march may run, against brute force."""
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rules") / "rules")
    csrc = os.path.join(ROOT, "paper_1008_0135_amd", "csrc")
    subprocess.check_call([HIPCC, "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", csrc,
                           os.path.join(HERE, "host", "rules_driver.cpp"), os.path.join(csrc, "plan.cpp"), "-o", exe],
                          stderr=subprocess.DEVNULL)

    def run(lines):
        text = "\n".join(" ".join(str(x) for x in line) for line in lines) + "\n"
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split()
        assert len(out) == len(lines)
        return [x == "1" for x in out]
    return run


def test_rows_readable(ask):
    """Windows of `pitch` floats a row over a box: the last float any of them reads."""
    rng = np.random.default_rng(3)
    lines, want = [], []
    for _ in range(400):
        n = rng.integers(2, 40, 3)
        lo = [int(rng.integers(0, k - 1)) for k in n]
        hi = [int(rng.integers(a + 1, k)) if rng.random() < 0.5 else int(k) - 1 for a, k in zip(lo, n)]
        pitch, tail = int(rng.choice([4, 8, 32, 64])), int(rng.choice([0, 64]))
        width = hi[0] - lo[0] + 1
        # a window starts at any column that keeps it inside the box, at the first if none does
        last = max((hi[2] * n[1] + hi[1]) * n[0] + f0 + pitch - 1
                   for f0 in range(lo[0], lo[0] + max(0, width - pitch) + 1))
        lines.append(["rows", *lo, *hi, *n, pitch, tail])
        want.append(bool(last < n[0] * n[1] * n[2] + tail))
    assert ask(lines) == want
    assert 50 < sum(want) < 380


def test_samples_countable(ask):
    """A float counter that is incremented by one reaches every count the rule lets pass."""
    assert np.float32(2 ** 24) + np.float32(1) == np.float32(2 ** 24)
    rng = np.random.default_rng(5)
    lines, counts = [], []
    for _ in range(300):
        lo = rng.integers(0, 5000, 3)
        ext = rng.integers(1, 4000, 3)
        step = float(2.0 ** rng.uniform(-18, 1))
        length = float(rng.choice([1.0, 0.25, 3.0]))  # parallel rays step by it
        lines.append(["count", *lo, *(lo + ext), repr(step), length])
        # most samples a ray along the diagonal can have in the box
        counts.append(int(np.sqrt(float((ext.astype(float) ** 2).sum())) / (step * length)) + 1)
    ok = ask(lines)
    assert all(c < 2 ** 24 for c, k in zip(counts, ok) if k)
    assert all(k for c, k in zip(counts, ok) if c < 0.999 * 2 ** 24)
    assert 30 < sum(ok) < 290
