"""The rule that sends multi-column products to the matrix cores (host)."""
import pytest

from tests.host_harness import run_cpp

FOUR, EIGHT, SIXTEEN = 1 << 2, 1 << 3, 1 << 4


@pytest.mark.parametrize("what,rows,patterns,slots,lanes,classes", [
    ("P1 elasticity", 3000, 1048, 130000, 1, FOUR | EIGHT | SIXTEEN),
    ("its rows cut by groups and rollers", 3000, 1300, 130000, 1, FOUR | EIGHT | SIXTEEN),
    ("Q1 elasticity, two lanes", 3000, 1050, 245000, 2, FOUR | EIGHT | SIXTEEN),
    ("P2 elasticity, one to eight lanes", 3000, 1100, 255000, 3.6, EIGHT | SIXTEEN),
    ("four lanes", 3000, 1100, 500000, 4, EIGHT | SIXTEEN),
    ("eight lanes", 3000, 1200, 600000, 8, 0),
    ("2-D elasticity, P1", 2000, 1000, 28000, 1, 0),
    ("two fields in space", 2000, 1000, 60000, 1, FOUR | EIGHT | SIXTEEN),
    ("with one condition on a node", 2000, 1001, 60000, 1, FOUR | EIGHT | SIXTEEN),
    ("with four lanes", 2000, 1010, 60000, 4, 0),
    ("one unknown per node", 2000, 2000, 60000, 1, 0),
    ("no rows", 0, 0, 0, 1, 0),
])
def test_tile_classes(tmp_path, what, rows, patterns, slots, lanes, classes):
    out = run_cpp(tmp_path, ["rules.h"], 'std::printf("%%d\\n", tile_classes(%s, %s, %s, %s));' % (
        float(rows), float(patterns), float(slots), float(lanes)))
    assert out == [str(classes)], what
