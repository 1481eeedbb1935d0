"""The benchmark names the Legendre kernels it runs: each is defined in the sources whose
hash decides whether a counter record still applies, and the records say which kernel of
those sources they were taken on."""
import json
import os
import re

import pytest

import bench

STAGES = [f"{d}_spin{s}" for d in ("m2a", "a2m") for s in (0, 2)]


def defined(family):
    text = ""
    for f in bench.LEG_SOURCES[family]:
        with open(os.path.join(bench.ROOT, f)) as fh:
            text += fh.read()
    return set(re.findall(r"__global__[^;{]*?\b(k_\w+)\s*\(", text))


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("stage", STAGES)
def test_launched_kernel_is_defined(stage, prec):
    name = bench.launched_kernel(stage, prec)
    assert re.match(r"\w+", name).group() in defined(bench.leg_family(name))


@pytest.mark.parametrize("path", [bench.TRAFFIC_FILE, bench.MFMA_FILE])
def test_records_name_their_kernel(path):
    with open(path) as fh:
        rec = json.load(fh)
    keys = {bench.record_key(s, p): bench.launched_kernel(s, p) for s in STAGES for p in ("fp64", "fp32", "bf16x3")}
    for key, e in rec.items():
        want, got = (re.match(r"\w+", x).group() for x in (keys[key], e["kernel"]))
        assert got == want, (key, e["kernel"])
