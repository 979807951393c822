"""The choice of kernel and tile for the bf16 matrix products, on the host, against the times of every form in
profiles/product_times.csv."""
import csv
import math
import os

import pytest

import paper_2502_00937_amd as V

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CACHE = 256 << 20  # the memory-side cache


def _table():
    with open(os.path.join(ROOT, "profiles", "product_times.csv")) as f:
        rows = list(csv.reader(line for line in f if not line.startswith("#")))
    assert rows[0][5:] == list(V.PRODUCT_FORMS)
    for r in rows[1:]:
        yield (r[0], int(r[3]), int(r[1]), int(r[2])), dict(zip(V.PRODUCT_FORMS, (float(t) if t else math.inf for t in r[5:])))


def _bytes(epilogue, rows, columns, depth):
    return rows * (2 * depth + columns * (2 if epilogue in ("bias", "gelu") else 4))


@pytest.mark.parametrize("past_cache", [False, True])
def test_the_form_chosen_is_near_the_best(past_cache):
    """How much longer than the best of the ten the chosen form took: on average 1.2 % where the memory-side cache holds operand
    and output, 0.2 % where it does not, at most 26 and 8 %.  Two runs of the table differ by 2.5 %, and single small products
    by 30, so the bars are wider than that.  Plans of two launches are left out: the table has no time of their parts."""
    logs = []
    for product, times in _table():
        form, rest, _, _ = V.vit_product_plan(*product)
        if rest == 0 and (_bytes(*product) > CACHE) == past_cache:
            assert times[form] < math.inf, product
            logs.append(math.log(times[form] / min(times.values())))
    assert len(logs) > 200
    assert sum(logs) / len(logs) < (0.01 if past_cache else 0.02)
    assert max(logs) < math.log(1.2 if past_cache else 1.35)


def test_a_device_of_few_units_takes_a_tile_per_workgroup():
    for product in (("bias", 150020, 3072, 1024), ("residual", 150020, 1024, 4096), ("patch", 149760, 384, 768)):
        assert V.vit_product_plan(*product)[0] == V.PRODUCT_FORMS[9]
        form, rest, _, _ = V.vit_product_plan(*product, units=255)
        assert form != V.PRODUCT_FORMS[9] and rest == 0
