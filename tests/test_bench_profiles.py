"""The counters that bench.py prints beside a measured time come from profiles/: only those taken of the kernel that
ran (the route it reports) may appear there.  Parity unpinned (own benchmark)."""
import json
import os

import pytest

import bench

PROFILES = os.path.join(bench.ROOT, "profiles")


@pytest.mark.parametrize("fname", ["traffic.json", "mfma_counters.json"])
def test_profiled_counters_only_beside_the_kernel_they_were_taken_of(fname):
    with open(os.path.join(PROFILES, fname)) as f:
        records = {k: v for k, v in json.load(f).items() if not k.startswith("_")}
    assert records
    for name, rec in records.items():
        def load(route):
            return bench.load_traffic(name, route) if fname == "traffic.json" else bench.load_mfma_counters(name, route, 100.0)

        assert load(rec["route"]) is not None
        for other in (rec["route"].replace("grid=", "grid=1"), "", None):
            assert load(other) is None, (name, other)


def test_profiled_kernels_are_those_of_their_routes():
    """<mode, row tiles, column tiles, waves, ring> of a per-tile kernel against the tile of its route."""
    for fname in ("traffic.json", "mfma_counters.json"):
        with open(os.path.join(PROFILES, fname)) as f:
            for name, rec in json.load(f).items():
                if name.startswith("_") or "gemm_prefill_dma_kernel" not in rec["kernel"]:
                    continue
                mode, mt, ct, waves, ring = rec["kernel"].split("<")[1].rstrip(">").split(", ")[:5]
                tile = "tile=%dx%d waves=%s ring=%s" % (32 * int(mt), 32 * int(ct) * int(waves), waves, ring)
                assert tile in rec["route"] and "mode=%s " % mode in rec["route"], (name, rec)
