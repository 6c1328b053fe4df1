"""Where one basis step of a constant operator is marched (march_rule.h, host
code): built with g++ and asked for grids whose step was timed both ways on one
MI355X.  The rule takes the faster way at each of them."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# operator, grid, element bytes, what the step also writes ("products", "ap" or
# nothing), us marched, us with a thread per point: of a step, or (above 700)
# of a solve with s = 9, whose last column is the one step
TIMED = [
    ("7", (187, 187, 187), 8, "ap", 44.9, 35.1), ("7", (187, 187, 187), 8, "", 35.2, 30.8),
    ("7", (187, 187, 187), 4, "ap", 24.9, 20.0), ("7", (200, 200, 200), 8, "ap", 50.8, 40.7),
    ("7", (200, 200, 200), 8, "", 38.3, 35.6), ("7", (224, 224, 224), 4, "ap", 40.2, 33.2),
    ("7", (225, 225, 225), 8, "ap", 75.4, 66.5), ("7", (256, 256, 256), 4, "ap", 63.5, 49.1),
    ("7", (256, 256, 256), 8, "", 72.5, 91.2), ("7", (400, 400, 400), 8, "ap", 468.3, 405.3),
    ("7", (1024, 1024, 3), 8, "ap", 22.3, 15.5), ("7", (2048, 2048, 16), 8, "ap", 482.1, 434.9),
    ("7", (1024, 1024, 8), 8, "", 41.1, 35.6), ("7", (1025, 1025, 8), 8, "", 40.9, 45.4),
    ("7", (601, 601, 64), 8, "", 104.2, 147.9), ("7", (31, 31, 8000), 8, "products", 58.9, 37.6),
    ("7", (300, 300, 300), 8, "products", 105.8, 168.9), ("7", (300, 300, 300), 4, "", 67.5, 79.7),
    ("7", (64, 200, 700), 4, "", 28.2, 25.9), ("7", (40, 40, 6000), 8, "ap", 61.6, 50.4),
    ("7", (147, 147, 147), 8, "products", 730.5, 774.1), ("7", (187, 187, 187), 8, "products", 1209.3, 1321.0),
    ("7", (40, 40, 6000), 8, "products", 1759.2, 1900.4), ("7", (1024, 1024, 3), 8, "products", 764.8, 802.7),
    ("7", (187, 187, 187), 4, "", 916.2, 933.0), ("7", (256, 256, 256), 4, "", 2354.6, 2406.4),
    ("27", (20, 20, 1500), 8, "ap", 14.0, 11.3), ("27", (32, 32, 600), 8, "products", 13.8, 11.1),
    ("27", (300, 8, 300), 8, "ap", 14.6, 12.9), ("27", (24, 24, 1500), 8, "products", 14.4, 15.8), ("27", (30, 200, 200), 4, "ap", 10.7, 9.6),
    ("27", (40, 40, 800), 4, "ap", 10.3, 9.7), ("27", (100, 100, 60), 8, "ap", 8.9, 12.0),
    ("27", (64, 64, 800), 8, "ap", 36.5, 48.6), ("27", (128, 128, 128), 4, "ap", 12.5, 16.4),
    ("27", (30, 400, 400), 4, "", 22.5, 37.0), ("27", (1024, 1024, 2), 8, "products", 16.8, 24.3),
]


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rule") / "march_rule_check")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-I",
                        os.path.join(ROOT, "paper_2512_09642_amd", "csrc"),
                        os.path.join(ROOT, "tests", "native", "march_rule_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def ask(rows):
        text = "".join(f"{d[0]} {d[1]} {d[2]} {int(op == '27')} {e} {int(w == 'products')} {int(w == 'ap')}\n"
                       for op, d, e, w in rows)
        return [int(v) for v in subprocess.run([exe], input=text, capture_output=True, text=True).stdout.split()]
    return ask


def test_the_faster_way(rule):
    got = rule([row[:4] for row in TIMED])
    assert len(got) == len(TIMED)
    for row, marched in zip(TIMED, got):
        assert marched == (row[4] < row[5]), row


def test_never_for_one_plane_or_few_unknowns(rule):
    rows = [(op, d, e, w) for op in ("7", "27") for e in (8, 4) for w in ("products", "ap", "")
            for d in ((2048, 2048, 1), (62, 30, 20), (1, 1, 2000000000), (2000000000, 1, 1), (1, 1, 1))]
    assert not any(rule(rows))
