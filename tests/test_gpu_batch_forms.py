"""The forms of a batch's XY pass, forced through the tuning file that a process reads (one child
process per form): the persistent launch and one launch per edge, at the edges worked by halves of
their planes in either, against the oracle and each other; and the tuner's report.

Every form gives the same bits.  Bars against the oracle: those of the batch's other tests, 1e-10 in
FP64, 1e-6 hartree and 2e-5 of xi in FP32."""

import os
import subprocess
import sys

import numpy as np
import pytest

import synth
from oracle import exchange

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
# (edge, orbitals): one transform (whole planes per edge) up to several hundred planes
SYSTEMS = {"c128": ((40, 3), (56, 3), (64, 1), (64, 2)), "c64": ((56, 2), (56, 3), (64, 1), (40, 2))}
H = 0.25

CHILD = """
import sys
import numpy as np, torch
sys.path.insert(0, sys.argv[1])
import paper_2405_01522_amd as ace
from tests import test_gpu_batch_forms as forms
out = {}
for name, dt in (("c128", torch.complex128), ("c64", torch.complex64)):
    b = ace.AceBatch(dt)
    systems = [{"h": forms.H, "phi": torch.from_numpy(p).to("cuda", dt)} for p in forms.orbitals(name)]
    b.build(systems)
    assert b.status()[0] == 0
    out[name + "_tuning"] = np.array(b.tuning())
    for k, s in enumerate(systems):
        for key in ("xi", "M", "ex"):
            out["%s_%d_%s" % (name, k, key)] = s[key].cpu().numpy()
np.savez(sys.argv[2], **out)
"""


def orbitals(name):
    single = name == "c64"
    return [synth.to_precision(synth.small_complex(900 + k, n, H, norb).phi, single)
            for k, (n, norb) in enumerate(SYSTEMS[name])]


def _run(tmp_path, form, cache):
    out = str(tmp_path / (form + ".npz"))
    env = dict(os.environ)
    env.pop("ACE_TUNE_CACHE", None)
    if cache:
        path = tmp_path / (form + ".txt")
        path.write_text("".join(line + "\n" for line in cache))
        env["ACE_TUNE_CACHE"] = str(path)
    res = subprocess.run([sys.executable, "-c", CHILD, ROOT, out], env=env, cwd=ROOT,
                         capture_output=True, text=True, timeout=100)
    assert res.returncode == 0, res.stderr[-3000:]
    return dict(np.load(out, allow_pickle=False))


def test_forms_agree(tmp_path):
    keys = {"c128": "dtype=0,edges=40-56-64", "c64": "dtype=1,edges=40-56-64"}
    shape = {"c128": "40:1:1024,56:1:1024,64:1:1024", "c64": "40:2:512,56:1:512,64:1:1024"}

    def lines(mode, zf, zi, xy=shape):
        return ["%s xy=%s mode=%s zf=%d zi=%d" % (keys[t], xy[t], mode, zf, zi) for t in keys]

    halves = {"c128": "40:1:0,56:1:0,64:1:0", "c64": "40:1:512,56:1:0,64:1:1024"}
    res = {"queue": _run(tmp_path, "queue", lines("queue", 512, 1024)),
           "edge": _run(tmp_path, "edge", lines("edge", 0, 0)),
           "edge, threads 0": _run(tmp_path, "edge0", lines("edge", 1024, 512, halves)),
           "tuned": _run(tmp_path, "tuned", None)}
    for form, r in res.items():
        for name in keys:
            t = str(r[name + "_tuning"])
            if form == "tuned":
                # FP64: 5 transforms at 40 (400 planes), 5 at 56, 3 at 64: all by halves;
                # FP32: 7 at 56 by halves, one at 64 not (128 planes), 40 never
                assert "source=tuned" in t
                assert ("40:1:0,56:1:0,64:1:0" if name == "c128" else "56:1:0,64:1:") in t, t
                assert name == "c128" or ("64:1:0" not in t and "40:1:0" not in t), t
            else:
                assert "source=cache" in t and "mode=" + form.split(",")[0] in t, t
            for key in res["queue"]:
                if key.startswith(name) and not key.endswith("tuning"):
                    assert np.array_equal(r[key], res["queue"][key]), (form, key)
    r = res["queue"]
    for name in keys:
        for k, phi in enumerate(orbitals(name)):
            xi, m, _, ex = exchange.ace_build(np.asarray(phi, dtype=np.complex128), H)
            got = [r["%s_%d_%s" % (name, k, key)] for key in ("xi", "M", "ex")]
            if name == "c128":
                assert abs(got[2] - ex) < 1e-10 * abs(ex)
                assert np.abs(got[0] - xi).max() < 1e-10 * np.abs(xi).max()
                assert np.abs(got[1] - m).max() < 1e-10 * np.abs(m).max()
            else:
                assert abs(got[2] - ex) < 1e-6
                assert np.abs(got[0] - xi).max() < 2e-5 * np.abs(xi).max()
