"""The autotuner's file: entries of earlier kernels are kept in it but not applied."""
import json
import re

import pytest

import synth
from gpu_common import dev, gal_inputs, soa

pytestmark = pytest.mark.gpu


def test_entries_of_earlier_kernels_are_timed_anew(filt6, tmp_path, monkeypatch):
    import paper_2506_19919_amd as sps
    path = tmp_path / "tune.json"
    monkeypatch.setenv("SPS_AUTOTUNE_CACHE", str(path))
    ctx = sps.Context(synth.ssp_grid(500), filt6, precisions=(sps.SPS_F32,), max_gal=300, max_exact=300)
    sfh, th, z = gal_inputs("dpl", 300, 891)
    args = (sfh, soa(th), dev(z))
    _, ms = ctx.autotune_exact(*args, prec=sps.SPS_F32)
    assert ms > 0
    (key, val), = json.loads(path.read_text()).items()
    # the same call's entry as it was written before the kernels had a number, with a choice of its own
    old = re.sub(r"\|kernels=\d+", "", key)
    other = dict(val, exact_order=1 if val["exact_order"] != 1 else 2)
    path.write_text('{\n  "%s": %s\n}\n' % (old, json.dumps(other)))
    ctx.set_launch(exact_order=0, exact_xcd=1, exact_ring=0)
    _, ms = ctx.autotune_exact(*args, prec=sps.SPS_F32)
    assert ms > 0                                          # timed, not taken from the old entry
    now = json.loads(path.read_text())
    assert now[old] == other and len(now) == 2             # which stays in the file
    _, ms = ctx.autotune_exact(*args, prec=sps.SPS_F32)
    assert ms == 0
    ctx.close()
