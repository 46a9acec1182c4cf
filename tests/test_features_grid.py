"""Workgroups of the feature product (CPU only, tests/host_features_grid.cpp).

A workgroup that takes all features of its pixels runs r^2 / 2 products in a
chain; where the pixels alone do not fill the chip (256 CUs) the features have
to be spread over workgroups too, and no grid may be empty or out of range."""
from host_cc import run_host


def test_few_pixels_still_fill_the_chip(tmp_path):
    run = run_host("host_features_grid.cpp", tmp_path)
    assert run.returncode == 0, run.stdout
    rows = [tuple(int(x) for x in line.split()) for line in run.stdout.splitlines()]
    assert len(rows) > 60
    for m, r, gx, gy, gz in rows:
        pieces = -(-m // 64) * -(-r // 16)            # 64 pixels x 16 features
        assert gz == 1 and 1 <= gx <= -(-m // 64) and 1 <= gy <= -(-r // 16) and gy <= 65535
        assert gx * gy >= min(pieces, 256), (m, r, gx, gy)
