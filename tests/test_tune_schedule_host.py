"""Whether a small 3D grid runs passes B, C and D in one launch is kept with its slab
count: written to the table file, read back, rejected where it cannot be, and absent
from files and hand-set entries that know nothing of it.  No GPU."""
import json

import pytest

from paper_2504_19410_amd import fsa as F

ROW = '{"precision": "f64", "grid": [12, 96, 8], "slabs": %s%s, "us": 20.0}'
DOC = '{"format": "fsa-tune-1", "arch": "", "entries": [], "schedules": [%s]}'


@pytest.fixture(autouse=True)
def clean_table():
    F.tune_reset()
    yield
    F.tune_reset()


def load(tmp_path, row):
    path = tmp_path / "in.json"
    path.write_text(DOC % row)
    F.tune_load(str(path))


@pytest.mark.parametrize("slabs,key,kept", [("1", ', "one_launch": 0', 0),
                                            ("1", ', "one_launch": 1', 1),
                                            ("4", ', "one_launch": 0', 0), ("1", "", None)])
def test_one_launch_survives_load_and_save(tmp_path, slabs, key, kept):
    load(tmp_path, ROW % (slabs, key))
    out = tmp_path / "out.json"
    F.tune_save(str(out))
    (row,) = json.loads(out.read_text())["schedules"]
    assert row["slabs"] == int(slabs) and row.get("one_launch") == kept
    F.tune_set_slabs("f64", (12, 96, 8), 1)    # by hand: nothing known
    F.tune_save(str(out))
    (row,) = json.loads(out.read_text())["schedules"]
    assert "one_launch" not in row


@pytest.mark.parametrize("slabs,key", [("1", ', "one_launch": 2'), ("1", ', "one_launch": -1'),
                                       ("1", ', "one_launch": 0.5'), ("2", ', "one_launch": 1')])
def test_impossible_rows_are_rejected(tmp_path, slabs, key):
    with pytest.raises(F.FsaError, match="EINVAL"):
        load(tmp_path, ROW % (slabs, key))
    assert F.tune_get_slabs("f64", (12, 96, 8)) == (1, 0.0)
