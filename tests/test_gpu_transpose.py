"""Transposed shards of every type pair, at any element address: whole tiles of
the tile kernel (fp32 128 x 256), register tiles (64 x 64 of 2-byte elements,
32 x 32 with fp32 on a side) whose last ones overlap, and blocks smaller than a
tile, packing and assembling, bit for bit against the oracle."""

import numpy as np
import pytest
import torch

import synthetic_checkpoint as sc
import paper_2609_25442_amd as wb
from oracle.catalog import CkptTensor
from oracle.layout import Layout, Local, Placement, RankLayout

from gpu_util import roundtrip, workspace_for
from wb_cases import to_wb

pytestmark = pytest.mark.gpu


def _values(catalog, dtype):
    return lambda t: sc.values_numpy(t, np.arange(catalog[t].numel), dtype).reshape(catalog[t].rows, catalog[t].cols)


@pytest.mark.parametrize("rows,cols,base,pad", [
    (1, 1, 0, 0), (31, 33, 1, 0), (32, 32, 0, 0), (64, 64, 0, 0), (63, 65, 0, 0), (65, 129, 3, 1), (100, 70, 2, 5),
    (256, 128, 0, 0), (260, 132, 0, 0), (513, 300, 0, 4), (300, 515, 1, 0), (257, 383, 0, 3)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_transposed_trainer(rows, cols, base, pad, dtype):
    """The trainer's shard holds T transposed (rows + pad elements a row, from
    element ``base``)."""
    cat = [CkptTensor("T", rows, cols)]
    tr = Layout(cat, [RankLayout([Local("t", dtype, 1, 1, base + cols * (rows + pad))],
                                 [Placement(0, 0, rows, 0, cols, 0, base, rows + pad, 1)])])
    ro = Layout(cat, [RankLayout([Local("x", dtype, 1, rows, cols)], [Placement(0, 0, rows, 0, cols, 0, 0, cols)])])
    p = wb.Plan(to_wb(tr), to_wb(ro), wb.SENDER, 0)
    es = 4 if dtype == "f32" else 2
    aligned = base * es % 16 == 0 and (rows + pad) * es % 16 == 0 and cols * es % 16 == 0
    assert p.launch_grid(4)[0] == ((cols // 128) * (rows // (1024 // es)) if aligned else 0)
    roundtrip(tr, ro, _values(cat, dtype), label=f"tr-{dtype}-{rows}x{cols}")


@pytest.mark.parametrize("tdt,rdt", [("bf16", "bf16"), ("f32", "f32"), ("f32", "bf16"), ("bf16", "f32")])
@pytest.mark.parametrize("ra,rb,cols", [(1, 31, 32), (32, 33, 64), (65, 66, 31), (128, 260, 256), (130, 71, 257), (129, 384, 512)])
def test_transposed_rollout(ra, rb, cols, tdt, rdt):
    """The rollout holds A and B transposed beside each other in one tensor."""
    cat = [CkptTensor("A", ra, cols), CkptTensor("B", rb, cols)]
    tr = Layout(cat, [RankLayout([Local("a", tdt, 1, ra, cols), Local("b", tdt, 1, rb, cols)],
                                 [Placement(0, 0, ra, 0, cols, 0, 0, cols), Placement(1, 0, rb, 0, cols, 1, 0, cols)])])
    W = ra + rb
    ro = Layout(cat, [RankLayout([Local("x", rdt, 1, cols, W)],
                                 [Placement(0, 0, ra, 0, cols, 0, 0, W, 1), Placement(1, 0, rb, 0, cols, 0, ra, W, 1)])])
    roundtrip(tr, ro, _values(cat, tdt), label=f"ro-{tdt}-{rdt}-{ra}+{rb}x{cols}")


@pytest.mark.parametrize("rows,cols", [(4096, 8192), (4096, 8448)])
def test_fp32_tiles_on_both_sides_of_the_cache_rule(rows, cols):
    """1024 tiles of 128 x 256 fp32 elements, the most that go without the
    non-temporal hint, and 1056."""
    L = wb.Layout.create([("T", rows, cols)], 1)
    L.add_local(0, "t", "f32", 1, rows, cols)
    L.add_placement(0, 0, 0, rows, 0, cols, 0, 0, cols)
    R = wb.Layout.create([("T", rows, cols)], 1)
    R.add_local(0, "x", "f32", 1, cols, rows)
    R.add_placement(0, 0, 0, rows, 0, cols, 0, 0, rows, 1)
    p = wb.Plan(L, R, wb.RECEIVER, 0)
    assert p.launch_grid(4)[0] == rows // 128 * (cols // 256)
    p.upload(workspace_for(p))
    x = torch.randn(rows, cols, device="cuda")
    out = wb.allocate_locals(R, 0)
    p.unpack(x.view(-1), out)
    torch.cuda.synchronize()
    assert torch.equal(out[0], x.t())
