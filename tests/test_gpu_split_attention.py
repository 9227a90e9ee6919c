"""GPU: the decode attention's segments (12 pages and more, at most 16 per row).

Calls with few (row, head) pairs spread a row's segments over workgroups, larger
calls keep a row in one workgroup; both must give the same bits, at contexts
around the page, class and segment edges.  The one-workgroup form is checked
against an fp32 softmax over the same bf16 cache: its output is rounded to bf16
(2^-9 relative) and its sums run in fp32 over at most 4000 positions."""
import sys

import numpy as np
import pytest
import torch

import cdbgen
import paper_2608_09444_amd as cdb
from test_gpu_edges import _batch_invariance, _own_pages

pytestmark = pytest.mark.gpu

# last positions: one token, page edges, the first segment's edge (12 pages = 192 tokens), several segments, the
# longest rows whose segments are still 12 pages (192 pages), longer segments
EDGES = (0, 15, 16, 63, 64, 190, 191, 192, 383, 384, 700, 3070, 3071, 3072, 3999)


def _shape(hd, H):
    return cdbgen.shrink(cdbgen.TINY, name=f"split-{H}x{hd}", d=H * hd, n_heads=H, head_dim=hd, d_ff=96,
                         n_prelude=0, n_core=2, n_coda=0)


def _rows(n, r_max):
    pos = np.zeros(n, np.int32)
    pos[:len(EDGES)] = EDGES
    idx = np.arange(n, dtype=np.int32)
    c = idx % r_max
    return {"slot": idx, "seq": idx.copy(), "pos": pos, "c": c.astype(np.int32),
            "depth": np.full(n, r_max, np.int32)}


@pytest.mark.parametrize("hd,H", [(64, 4), (96, 3), (128, 2)])
def test_segments_over_workgroups_give_the_same_bits(hd, H):
    s = _shape(hd, H)
    n = 320 // H + (320 % H > 0)  # the smallest batch that keeps rows in one workgroup
    rows = _rows(n, s.r_max)
    print(f"[gpu] split attention {H} x {hd}: {n} rows vs their first {len(EDGES)}", flush=True)
    sys.stdout.flush()
    _batch_invariance(s, cdbgen.model_weights(s), rows, len(EDGES))


@pytest.mark.parametrize("hd,H", [(64, 4), (96, 3), (128, 2)])
def test_one_workgroup_form_against_fp32(hd, H):
    s = _shape(hd, H)
    rows_np = _rows(len(EDGES), s.r_max)
    pt, max_pages, n_pages = _own_pages(s, rows_np)
    kv = cdb.PagedKV(s, len(EDGES), max_pages, 0, n_pages, 0, fill="random")
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    kv.core.normal_(0.0, 1.0, generator=g)
    kv.page_table.copy_(torch.from_numpy(pt))
    rows = cdb.Rows(rows_np["slot"], rows_np["seq"], rows_np["pos"], rows_np["c"], rows_np["depth"])
    q = torch.empty((len(EDGES), s.d), device="cuda").normal_(0.0, 1.0, generator=g)
    out = torch.zeros((32, s.d), dtype=torch.bfloat16, device="cuda")
    ws = torch.zeros(256 + 4 * 256, dtype=torch.uint8, device="cuda")
    print(f"[gpu] paged attention {H} x {hd}", flush=True)
    cdb.cdb_paged_attention(cdb.make_desc(s), kv.c, rows.c, 1, 1, q, out, ws)
    torch.cuda.synchronize()
    assert cdb.cdb_read_device_error(ws) == 0
    # fragment order -> [row][d]
    got = out.view(s.d // 16, 2, 32, 8).permute(2, 0, 1, 3).reshape(32, s.d)[:len(EDGES)].float().cpu()
    core = kv.core.float().cpu()
    for i, p in enumerate(EDGES):
        pids = pt[i, int(rows_np["c"][i]) + 1, :p // 16 + 1]
        k, v = (core[1, pids, t].permute(1, 0, 2, 3).reshape(H, -1, hd)[:, :p + 1] for t in (0, 1))
        qi = q[i].cpu().view(H, 1, hd)
        pr = torch.softmax((qi * k).sum(-1) / hd ** 0.5, -1)
        want = (pr[..., None] * v).sum(1).reshape(-1)
        err = (got[i] - want).abs()
        assert bool((err <= want.abs() * 2.0 ** -8 + 1e-4).all()), (p, float(err.max()))
