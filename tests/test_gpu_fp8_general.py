"""The fp8 block kernel's path for blocks that are no aligned bf16 piece: fp32
sources (a correctly rounded quotient without a division), sources at any
element address, widths that are no multiple of a chunk, blocks cut by columns
or in the middle of a row, and blocks of mixed wire types."""

import numpy as np
import pytest
import torch

import synthetic_checkpoint as sc
import paper_2609_25442_amd as wb
from oracle import casts
from oracle.catalog import CkptTensor
from oracle.layout import Layout, Local, Placement, RankLayout

from gpu_util import roundtrip, workspace_for

pytestmark = pytest.mark.gpu


def _values(catalog, dtype):
    return lambda t: sc.values_numpy(t, np.arange(catalog[t].numel), dtype).reshape(catalog[t].rows, catalog[t].cols)


def _trainer(cat, how, dtype):
    c = cat[0]
    if how == "whole":
        return Layout(cat, [RankLayout([Local("t", dtype, 1, c.rows, c.cols)], [Placement(0, 0, c.rows, 0, c.cols, 0, 0, c.cols)])])
    if how == "columns":
        m = max(1, c.cols // 2 - 1)
        cuts = [(0, m), (m, c.cols)]
        return Layout(cat, [RankLayout([Local("t", dtype, 1, c.rows, b - a)], [Placement(0, 0, c.rows, a, b, 0, 0, b - a)])
                            for a, b in cuts if a < b])
    # flat shards that end in the middle of a row
    ranks, n = [], c.numel
    cuts = [0, n // 3 + 1, 2 * n // 3 + 2, n]
    for a, b in zip(cuts, cuts[1:]):
        pls, p = [], a
        while p < b:
            r, k = divmod(p, c.cols)
            rows = (b - p) // c.cols if k == 0 else 0
            if rows:
                pls.append(Placement(0, r, r + rows, 0, c.cols, 0, p - a, c.cols))
                p += rows * c.cols
            else:
                w = min(b - p, c.cols - k)
                pls.append(Placement(0, r, r + 1, k, k + w, 0, p - a, c.cols))
                p += w
        ranks.append(RankLayout([Local("t", dtype, 1, 1, b - a)], pls))
    return Layout(cat, ranks)


def _rollout(cat, block):
    c = cat[0]
    return Layout(cat, [RankLayout([Local("q", "f8e4m3", 1, c.rows, c.cols, block, scale=1),
                                    Local("s", "f32", 1, -(-c.rows // block), -(-c.cols // block), scales=0)],
                                   [Placement(0, 0, c.rows, 0, c.cols, 0, 0, c.cols)])])


@pytest.mark.parametrize("how", ["whole", "columns", "flat"])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("rows,cols,block", [(300, 264, 128), (300, 261, 128), (129, 130, 128), (130, 131, 128), (70, 3, 128),
                                             (9, 5, 4), (140, 67, 64), (65, 33, 32), (33, 17, 16), (260, 128, 128)])
def test_general_blocks(how, dtype, rows, cols, block):
    cat = [CkptTensor("T", rows, cols)]
    roundtrip(_trainer(cat, how, dtype), _rollout(cat, block), _values(cat, dtype), label=f"{how}-{dtype}-{rows}x{cols}/{block}")


def test_mixed_wire_types_in_one_block():
    """One rank ships its columns as fp32, the other as bf16: blocks with both
    divide by IEEE division, element by element."""
    rows, cols, m = 200, 200, 70
    L = wb.Layout.create([("T", rows, cols)], 2)
    L.add_local(0, "a", "f32", 1, rows, m)
    L.add_placement(0, 0, 0, rows, 0, m, 0, 0, m)
    L.add_local(1, "b", "bf16", 1, rows, cols - m)
    L.add_placement(1, 0, 0, rows, m, cols, 0, 0, cols - m)
    R = wb.Layout.create([("T", rows, cols)], 1)
    R.add_local(0, "q", "f8e4m3", 1, rows, cols, 128)
    R.add_placement(0, 0, 0, rows, 0, cols, 0, 0, cols)
    p = wb.Plan(L, R, wb.RECEIVER, 0)
    p.upload(workspace_for(p))
    x = (torch.randn(rows, cols, generator=torch.Generator().manual_seed(5)) * 0.02)
    x[:, m:] = x[:, m:].bfloat16().float()
    recv = torch.zeros(p.buffer_bytes, dtype=torch.uint8, device="cuda")
    for s, (a, b, dt) in enumerate([(0, m, torch.float32), (m, cols, torch.bfloat16)]):
        _, off, nb = p.region(s, 0)
        recv[off:off + nb] = x[:, a:b].to(dt).contiguous().view(-1).view(torch.uint8).cuda()
    q = torch.zeros(rows, cols, dtype=torch.float8_e4m3fn, device="cuda")
    s = torch.zeros(2, 2, dtype=torch.float32, device="cuda")
    p.unpack(recv, [q, s])
    codes, scales = casts.quantize_matrix(x.numpy(), 128)
    assert np.array_equal(q.view(torch.uint8).cpu().numpy(), codes)
    assert np.array_equal(s.cpu().numpy(), scales)


def _grid(rows, cols, h, w):
    return [(r, min(rows, r + h), c, min(cols, c + w)) for r in range(0, rows, h) for c in range(0, cols, w)]


@pytest.mark.parametrize("rows,cols,h,w", [(200, 264, 30, 264), (200, 261, 7, 261), (140, 130, 140, 13), (130, 131, 61, 45),
                                           (128, 128, 4, 16), (128, 128, 1, 64), (129, 127, 5, 8), (40, 6, 3, 6)])
def test_mixed_wire_types_however_cut(rows, cols, h, w):
    """Pieces of h rows by w columns, by turns fp32 and bf16 (a rank each): bands,
    chunks that straddle pieces, ragged edges and more pieces than are staged."""
    parts = _grid(rows, cols, h, w)
    dts = ["f32" if (i + i // -(-cols // w)) % 2 else "bf16" for i in range(len(parts))]
    L = wb.Layout.create([("T", rows, cols)], len(parts))
    for i, ((r0, r1, c0, c1), dt) in enumerate(zip(parts, dts)):
        L.add_local(i, "t", dt, 1, r1 - r0, c1 - c0)
        L.add_placement(i, 0, r0, r1, c0, c1, 0, 0, c1 - c0)
    R = wb.Layout.create([("T", rows, cols)], 1)
    R.add_local(0, "q", "f8e4m3", 1, rows, cols, 128)
    R.add_placement(0, 0, 0, rows, 0, cols, 0, 0, cols)
    p = wb.Plan(L, R, wb.RECEIVER, 0)
    p.upload(workspace_for(p))
    x = torch.randn(rows, cols, generator=torch.Generator().manual_seed(rows)) * 0.02
    recv = torch.full((p.buffer_bytes,), 0x7F, dtype=torch.uint8)
    for i, ((r0, r1, c0, c1), dt) in enumerate(zip(parts, dts)):
        piece = x[r0:r1, c0:c1].to(torch.bfloat16 if dt == "bf16" else torch.float32).contiguous()
        x[r0:r1, c0:c1] = piece.float()
        _, off, nb = p.region(i, 0)
        recv[off:off + nb] = piece.view(-1).view(torch.uint8)
    q = torch.zeros(rows, cols, dtype=torch.float8_e4m3fn, device="cuda")
    s = torch.zeros(-(-rows // 128), -(-cols // 128), dtype=torch.float32, device="cuda")
    p.unpack(recv.cuda(), [q, s])
    codes, scales = casts.quantize_matrix(x.numpy(), 128)
    assert np.array_equal(s.cpu().numpy(), scales)
    assert np.array_equal(q.view(torch.uint8).cpu().numpy(), codes)


def test_f32_quotients_next_to_rounding_boundaries():
    """fp32 sources whose quotients lie within a few ulps of every E4M3 rounding
    boundary (midpoints of neighbouring values), over block maxima of every
    exponent the correction steps and the division share, of random
    significands and of the one they exclude (s all ones), against IEEE
    division: the codes are the same, whichever form a block takes."""
    nb = 4096
    rows = nb * 128
    cat = [("X", rows, 128)]
    tr = wb.Layout.create(cat, 1)
    tr.add_local(0, "x", "f32", 1, rows, 128)
    tr.add_placement(0, 0, 0, rows, 0, 128, 0, 0, 128)
    ro = wb.Layout.create(cat, 1)
    ro.add_local(0, "y", "f8e4m3", 1, rows, 128, 128)
    ro.add_placement(0, 0, 0, rows, 0, 128, 0, 0, 128)
    p = wb.Plan(tr, ro, wb.RECEIVER, 0)
    p.upload(workspace_for(p))
    g = torch.Generator(device="cuda").manual_seed(11)
    e = torch.randint(-100, 112, (nb,), generator=g, device="cuda")
    amax = torch.ldexp(1 + torch.rand(nb, generator=g, device="cuda"), e)
    ones = torch.ldexp(torch.full((nb // 8,), 2.0 - 2.0 ** -23, device="cuda"), e[:nb // 8]) * 448.0  # s close to all ones
    amax[:nb // 8] = (ones.view(torch.int32) + torch.arange(nb // 8, device="cuda", dtype=torch.int32) % 5 - 2).view(torch.float32)
    s = amax / torch.full_like(amax, 448.0)
    assert bool(((s.view(torch.int32) & 0x7FFFFF) == 0x7FFFFF).any())
    v = torch.from_numpy(casts.E4M3_VALUES.astype(np.float32)).cuda()
    mid = torch.cat([(v[1:] + v[:-1]) / 2, v[1:-1]])                       # boundaries, and values themselves
    k = torch.randint(0, mid.numel(), (nb, 16384), generator=g, device="cuda")
    x = mid[k] * s[:, None]
    off = torch.randint(-3, 4, (nb, 16384), generator=g, device="cuda", dtype=torch.int32)
    x = (x.view(torch.int32) + off).view(torch.float32)
    x = torch.minimum(x, amax[:, None])
    x[:, 1::2] = -x[:, 1::2]
    at = torch.randint(0, 16384, (nb,), generator=g, device="cuda")
    x[torch.arange(nb, device="cuda"), at] = amax
    q = torch.empty(rows, 128, dtype=torch.float8_e4m3fn, device="cuda")
    sc_ = torch.empty(nb, 1, dtype=torch.float32, device="cuda")
    p.unpack(x.contiguous(), [q, sc_])
    assert torch.equal(sc_.view(-1), s)
    want = (x / s[:, None]).to(torch.float8_e4m3fn).view(torch.uint8)
    bad = torch.nonzero(q.view(torch.uint8).view(nb, -1) != want)
    assert bad.numel() == 0, (bad.shape[0], bad[:5].tolist())
