"""Copies and casts whose rows sit at any element address: packing from shards
that start anywhere with a pitch of their own, assembling into columns of a
wider tensor, at widths around the kernel's units (4 or 8 elements), chunks
(64 units) and work items, bit for bit against the oracle."""

import numpy as np
import pytest

import synthetic_checkpoint as sc
import paper_2609_25442_amd as wb
from oracle.catalog import CkptTensor
from oracle.layout import Layout, Local, Placement, RankLayout

from gpu_util import roundtrip
from wb_cases import to_wb

pytestmark = pytest.mark.gpu


def _values(catalog, dtype):
    return lambda t: sc.values_numpy(t, np.arange(catalog[t].numel), dtype).reshape(catalog[t].rows, catalog[t].cols)


def _layouts(rows, wa, wb_, base, pad, tdt, rdt):
    """A [rows, wa] and B [rows, wb_]: the trainer holds each in a padded
    buffer from element ``base`` with rows of width + pad; the rollout holds
    them side by side in one tensor."""
    cat = [CkptTensor("A", rows, wa), CkptTensor("B", rows, wb_)]
    loc, pl = [], []
    for t, w in enumerate((wa, wb_)):
        loc.append(Local("t%d" % t, tdt, 1, 1, base + rows * (w + pad)))
        pl.append(Placement(t, 0, rows, 0, w, t, base, w + pad))
    tr = Layout(cat, [RankLayout(loc, pl)])
    W = wa + wb_
    ro = Layout(cat, [RankLayout([Local("x", rdt, 1, rows, W)],
                                 [Placement(0, 0, rows, 0, wa, 0, 0, W), Placement(1, 0, rows, 0, wb_, 0, wa, W)])])
    return cat, tr, ro


@pytest.mark.parametrize("tdt,rdt", [("bf16", "bf16"), ("f32", "f32"), ("f32", "bf16"), ("bf16", "f32")])
@pytest.mark.parametrize("rows,wa,wb_,base,pad", [
    (1, 3, 4, 1, 0), (3, 5, 7, 1, 1), (5, 8, 9, 3, 2), (7, 4, 15, 0, 1), (2, 16, 17, 7, 0), (130, 63, 66, 5, 3),
    (33, 511, 514, 1, 0), (9, 1024, 1025, 8, 8), (257, 96, 104, 8, 8), (1, 70001, 131075, 1, 0), (3, 65537, 140003, 2, 5),
    (40, 1721, 1500, 11, 0), (1, 10004, 65540, 4, 0), (1, 131072, 70001, 8, 0), (1, 8191, 8192, 8, 0),
    (1, 8196, 100012, 12, 0)])
def test_rows_at_any_element(rows, wa, wb_, base, pad, tdt, rdt):
    cat, tr, ro = _layouts(rows, wa, wb_, base, pad, tdt, rdt)
    roundtrip(tr, ro, _values(cat, tdt), label=f"rows-{rows}x{wa}+{wb_}-{base}-{pad}-{tdt}-{rdt}")


@pytest.mark.parametrize("task_bytes", [1024, 1 << 20])
def test_row_items_of_other_sizes(task_bytes, monkeypatch):
    monkeypatch.setenv("WB_TASK_BYTES", str(task_bytes))
    cat, tr, ro = _layouts(19, 517, 4099, 3, 2, "f32", "bf16")
    roundtrip(tr, ro, _values(cat, "f32"), label=f"row-items-{task_bytes}")


def test_row_items_are_no_longer_than_aligned_ones():
    """An unaligned run is cut so that its items need no more workgroups each
    than aligned ones: every item of a launch gets as many as its longest."""
    for tdt, rdt in (("bf16", "bf16"), ("f32", "bf16"), ("bf16", "f32"), ("f32", "f32")):
        per_item = []
        for base in (0, 1):
            n = 1 << 22
            cat = [CkptTensor("A", 1, n)]
            tr = Layout(cat, [RankLayout([Local("t", tdt, 1, 1, n)], [Placement(0, 0, 1, 0, n, 0, 0, n)])])
            ro = Layout(cat, [RankLayout([Local("x", rdt, 1, 1, n + base), ],
                                         [Placement(0, 0, 1, 0, n, 0, base, n)] +
                                         ([Placement(0, 0, 1, 0, 1, 0, 0, 1)] if base else []))])
            p = wb.Plan(to_wb(tr), to_wb(ro), wb.RECEIVER, 0)
            x, y, _ = p.launch_grid(0)
            per_item.append(x * y / (p.work_counts()[0] - base))
        assert per_item[1] <= per_item[0] * 1.01, (tdt, rdt, per_item)
