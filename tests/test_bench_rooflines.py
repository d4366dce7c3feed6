"""bench.py's install records, from counters alone (no GPU): launches that
read the ring count against HBM, launches that read pinned memory against the
host link, and neither has the other's time or bytes."""

import pytest

import bench


def _stats(ring, direct):
    (rn, rb, rms), (dn, db, dms) = ring, direct
    return {"n_install_launches": rn + dn, "installed_bytes": rb + db, "install_ms_total": rms + dms,
            "direct": {"n_launches": dn, "bytes": db, "ms_total": dms}}


@pytest.mark.parametrize("ring,direct", [((4, 4_000_000_000, 1.25), (0, 0, 0.0)), ((0, 0, 0.0), (8, 600_000_000, 11.0)),
                                         ((2, 2_000_000_000, 0.625), (3, 300_000_000, 5.5))])
def test_each_install_kernel_has_its_own_record(ring, direct):
    a, b = bench.install_rooflines([_stats(ring, direct)] * 3, 57.0)
    assert (a is None) == (ring[0] == 0) and (b is None) == (direct[0] == 0)
    if a:
        assert (a["kernel"], a["bound"], a["launches_timed"]) == ("k_install", "hbm", 3 * ring[0])
        assert a["bytes_per_launch"] == 2 * ring[1] // ring[0] and a["achieved"] == pytest.approx(6400.0)
    if b:
        assert (b["kernel"], b["bound"], b["launches_timed"]) == ("k_install_direct", "host link", 3 * direct[0])
        assert b["bytes_per_launch"] == direct[1] // direct[0]
        assert b["achieved"] == pytest.approx(54.5, abs=0.1) and b["frac_of_measured_link"] == pytest.approx(0.957, abs=2e-3)
