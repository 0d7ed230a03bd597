"""The rules that choose the products' forms (host)."""
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


F64, F32, BF16 = 1, 2, 4
ALL = F64 | F32 | BF16


@pytest.mark.parametrize("what,widest,columns,slots,rows,patterns,vec,lines,forms", [
    ("P1 elasticity", 400, 9e5, 9e6, 2e5, 7e4, 2, 8.5, ALL),
    ("P1 elasticity in runs", 400, 9e5, 9e6, 2e5, 7e4, 2, 5, ALL),
    ("P1 Laplacian", 300, 4e5, 1e6, 7e4, 7e4, 1, 5, ALL),
    ("Q1 Laplacian", 300, 4e5, 1e6, 4e4, 4e4, 2, 8, ALL),
    ("in natural numbering", 300, 4e5, 1e6, 4e4, 4e4, 2, 7, F64 | F32),
    ("45 % of the slots", 300, 4.5e5, 1e6, 7e4, 7e4, 2, 64, ALL),
    ("over it", 300, 4.6e5, 1e6, 7e4, 7e4, 2, 64, 0),
    ("rows of their own, 32 KB of LDS", 1023, 1e5, 1e6, 2e4, 2e4, 2, 64, ALL),
    ("over it", 1024, 1e5, 1e6, 2e4, 2e4, 2, 64, F32 | BF16),
    ("shared rows", 1280, 1e5, 1e6, 2e4, 1e4, 2, 64, ALL),
    ("over the limit", 1281, 1e5, 1e6, 2e4, 1e4, 2, 64, 0),
])
def test_stage_forms(tmp_path, what, widest, columns, slots, rows, patterns, vec, lines, forms):
    out = run_cpp(tmp_path, ["rules.h"], 'std::printf("%%d\\n", stage_forms(%d, %s, %s, %s, %s, %d, %s));' % (
        widest, float(columns), float(slots), float(rows), float(patterns), vec, lines * slots / 64))
    assert out == [str(forms)], what


@pytest.mark.parametrize("slots,f32", [(1.06e7, True), (1.07e7, False), (2.99e7, False), (3.01e7, True)])
@pytest.mark.parametrize("what,rows_per_pattern,vec,lines", [
    ("runs of neighbours", 1, 2, 5.5), ("rows that share columns", 3, 2, 5.5), ("single slots", 1, 1, 5.5), ("no runs", 1, 2, 8)])
def test_float_products_of_runs(tmp_path, what, rows_per_pattern, vec, lines, slots, f32):
    """FP32 products of runs of neighbours gather per slot from 64 to 180 MB
    of slots, the others never for that."""
    out = run_cpp(tmp_path, ["rules.h"], 'std::printf("%%d\\n", stage_forms(300, %s, %s, %s, %s, %d, %s));' % (
        0.35 * slots, slots, slots / 27, slots / 27 / rows_per_pattern, vec, lines * slots / 64))
    runs = what == "runs of neighbours"
    assert out == [str(F64 | (0 if runs else BF16) | (F32 if f32 or not runs else 0))], what


def test_rows_too_short_to_stage(tmp_path):
    out = run_cpp(tmp_path, ["rules.h"], r"""
    for (int w : {1, 3, 4, 5, 7}) std::printf("%d ", int(stage_pays(64.0 * w, 64.0)));
""")
    assert out == ["0", "0", "0", "1", "1"]


def test_workgroup_choice_is_kept_per_kernel(tmp_path):
    """Batches of the same totals, of which one holds its slots in registers,
    are timed apart."""
    out = run_cpp(tmp_path, ["rules.h"], r"""
    const WgKey a = wg_key(0, 300, 634800, 4400000, 9, 7, true), b = wg_key(0, 300, 634800, 4400000, 9, 7, false);
    std::printf("%d %d\n", int(a == b), int(a == wg_key(0, 300, 634800, 4400000, 9, 7, true)));
""")
    assert out == ["0", "1"]
