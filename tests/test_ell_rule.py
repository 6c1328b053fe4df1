"""Which sliced CSR matrices go through the caches (ell_rule.h, host code): built
with g++ and asked for matrices whose basis step was timed both ways on one
MI355X.  The rule takes the faster way at each of them."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# rows, entries of a slice's longest row, rows its columns reach over, bytes of a
# value, us cached, us non-temporal
TIMED = [
    (500000, 14, 500000, 8, 31.28, 34.71), (600000, 14, 600000, 8, 41.41, 42.05), (750000, 13, 750000, 8, 52.50, 49.32),
    (1000000, 14, 1000000, 8, 86.48, 81.27), (1500000, 9, 1500000, 8, 76.33, 73.17), (2000000, 8, 2000000, 8, 85.50, 82.56),
    (500000, 14, 500000, 4, 22.44, 27.07), (1000000, 14, 1000000, 4, 47.66, 54.09), (1500000, 9, 1500000, 4, 49.27, 48.51),
    (2000000, 8, 2000000, 4, 60.65, 58.61), (300000, 14, 300000, 8, 18.9, 21.87),
    (1000000, 7, 20500, 8, 19.65, 23.75), (2000376, 7, 32300, 8, 32.80, 44.84), (2000376, 7, 32300, 4, 26.50, 32.30),
    (1030301, 7, 0, 8, 15.2, 17.5), (7077888, 7, 0, 8, 126.0, 109.0),
]


def test_the_faster_way(tmp_path):
    exe = str(tmp_path / "ell_rule_check")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-I",
                        os.path.join(ROOT, "paper_2512_09642_amd", "csrc"),
                        os.path.join(ROOT, "tests", "native", "ell_rule_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    text = "".join(f"{n * w} {span} {elem}\n" for n, w, span, elem, _, _ in TIMED)
    got = [int(v) for v in subprocess.run([exe], input=text, capture_output=True, text=True).stdout.split()]
    assert len(got) == len(TIMED)
    for row, kept in zip(TIMED, got):
        assert kept == (row[4] < row[5]), row
