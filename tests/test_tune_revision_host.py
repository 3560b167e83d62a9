"""Variants 0 and 2 of the fused pass's two-wave teams (FP32 768, 1536, 2048, FP64 2048)
changed places after tables had been saved: a file of revision 1 (or none) names the
shape it measured, not the number.  Everywhere else, and in files of the present
revision, the number stands.  No GPU."""
import json
import os

import pytest

from paper_2504_19410_amd import fsa as F

DOC = ('{"format": "fsa-tune-1", %s"arch": "", "entries": [{"precision": "%s", "pass": "%s", '
       '"length": %d, "class": 10, "variant": %d, "occupancy": 1, "us": 9.0}]}')


@pytest.fixture(autouse=True)
def clean_table():
    F.tune_reset()
    yield
    F.tune_reset()


@pytest.mark.parametrize("prec,name,length,var,want", [
    ("f32", "conv", 2048, 2, 0), ("f32", "conv", 2048, 0, 2), ("f32", "conv", 2048, 1, 1),
    ("f32", "conv", 768, 2, 0), ("f32", "conv", 1536, 0, 2), ("f64", "conv", 2048, 2, 0),
    ("f32", "batched_conv", 2048, 0, 2),
    # one-wave and four-wave teams, FP64 of 3 * 2^a, the other passes
    ("f32", "conv", 512, 2, 2), ("f64", "conv", 768, 2, 2), ("f64", "conv", 1536, 0, 0),
    ("f32", "conv", 1024, 2, 2), ("f32", "r2c", 768, 2, 2), ("f32", "fwd_t", 2048, 0, 0),
])
def test_old_files_name_the_shape(tmp_path, prec, name, length, var, want):
    path = tmp_path / "t.json"
    for head, expect in (("", want), ('"revision": 1, ', want), ('"revision": 2, ', var)):
        F.tune_reset()
        path.write_text(DOC % (head, prec, name, length, var))
        F.tune_load(str(path))
        assert F.tune_get(prec, name, length, 1024)[:2] == (expect, 1), head


def test_a_saved_file_reads_back_as_it_was(tmp_path):
    F.tune_set("f32", "conv", 2048, 2, 0, 1024)
    path = tmp_path / "t.json"
    F.tune_save(str(path))
    assert json.loads(path.read_text())["revision"] == 2
    F.tune_reset()
    F.tune_load(str(path))
    assert F.tune_get("f32", "conv", 2048, 1024)[0] == 2


def test_unknown_revisions_are_rejected_and_the_shipped_table_is_current(tmp_path):
    path = tmp_path / "t.json"
    path.write_text(DOC % ('"revision": 3, ', "f32", "conv", 512, 0))
    with pytest.raises(F.FsaError, match="EINVAL"):
        F.tune_load(str(path))
    shipped = os.path.join(os.path.dirname(F.__file__), "tune", "gfx950.json")
    with open(shipped) as f:
        assert json.load(f)["revision"] == 2
