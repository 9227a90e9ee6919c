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


def _step_bits(s, rows_np, calls, unmap=None, captured=False):
    """Loop steps of the first `capacity` rows, `live` of them counted on the device (None: the host's count), one
    after the other on one workspace from the same state and cache: [(states, scores, error code)].  unmap: a (row,
    page) whose entry in the page table is -1.  captured: calls with a device count are replays of one graph per
    capacity, captured at its first call (after an eager one, which sets the kernels' attributes)."""
    n = len(rows_np["pos"])
    gm = cdb.DeviceModel(s, cdbgen.model_weights(s))
    pt, max_pages, n_pages = _own_pages(s, rows_np)
    if unmap is not None:
        pt[unmap[0], int(rows_np["c"][unmap[0]]) + 1, unmap[1]] = -1
    kv = cdb.PagedKV(s, n, max_pages, 0, n_pages, 0, fill="random")
    g = torch.Generator(device="cuda")
    g.manual_seed(22)
    kv.core.normal_(0.0, 1.0, generator=g)
    kv.page_table.copy_(torch.from_numpy(pt))
    state = cdb.State(s, n)
    state.h.normal_(0.0, 1.0, generator=g)
    if s.injection:
        state.e.normal_(0.0, 1.0, generator=g)
    h0 = state.h.clone()
    ws = cdb.Workspace(gm.desc, n)
    got, graphs = [], {}
    for capacity, live in calls:
        print(f"[gpu]   {capacity} rows, {live} live", flush=True)
        replay = captured and live is not None
        if replay and capacity in graphs:
            graph, count, rows, out = graphs[capacity]
            count.fill_(live)
        else:
            count = None if live is None else torch.tensor([live], dtype=torch.int32, device="cuda")
            rows = cdb.Rows(*(rows_np[k][:capacity] for k in ("slot", "seq", "pos", "c", "depth")), d_n_rows=count)
            out = cdb.StepOut(capacity)
        if replay and capacity not in graphs:
            cdb.cdb_loop_step(gm.model, kv.c, state.c, rows.c, out.c, ws.buf)
            torch.cuda.synchronize()
            graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
            with torch.cuda.graph(graph, stream=side):
                cdb.cdb_loop_step(gm.model, kv.c, state.c, rows.c, out.c, ws.buf, stream=side)
            torch.cuda.synchronize()
            graphs[capacity] = graph, count, rows, out
        state.h.copy_(h0)
        torch.cuda.synchronize()
        if replay:
            graph.replay()
        else:
            cdb.cdb_loop_step(gm.model, kv.c, state.c, rows.c, out.c, ws.buf)
        torch.cuda.synchronize()
        got.append((state.h.clone(), out.score.clone(), cdb.cdb_read_device_error(ws.buf)))
    return h0, got


# 16 heads: a row's segments over several workgroups below 20 rows (4 workgroups at 19 rows, so each takes several
# segments of the long rows), row pairs up to 64 rows (512 pairs), one workgroup per row above; the device count chooses
# between the last two
@pytest.mark.parametrize("hd,captured", [(64, False), (96, False), (128, False), (128, True)])
def test_every_form_and_device_count_gives_the_same_bits(hd, captured):
    s = _shape(hd, 16)
    rows = _rows(67, s.r_max)
    rows["pos"][len(EDGES):] = np.random.default_rng(6).integers(0, 1200, 67 - len(EDGES))
    calls = [(67, None), (66, None), (65, None), (64, None), (20, None), (19, None), (67, 67), (67, 65), (67, 64),
             (67, 20), (67, 1), (19, 19), (19, 15), (19, 7), (19, 1), (19, 0), (19, 15)]
    print(f"[gpu] attention forms 16 x {hd}, captured {captured}", flush=True)
    h0, got = _step_bits(s, rows, calls, captured=captured)
    h, score, _ = got[0]
    for (capacity, live), (hc, sc, err) in zip(calls, got):
        m = capacity if live is None else live
        assert err == 0
        assert torch.equal(hc[:m], h[:m]) and torch.equal(sc[:m], score[:m]), (capacity, live)
        assert torch.equal(hc[m:], h0[m:]), (capacity, live)


def test_unmapped_page_in_every_form():
    """An unmapped page inside a long row's context is reported and left out, alike in the three forms, and reaches no
    other row."""
    s = _shape(64, 16)
    rows = _rows(66, s.r_max)
    row = EDGES.index(3071)
    calls = [(66, None), (64, None), (19, None), (19, 15)]
    print("[gpu] attention forms, an unmapped page", flush=True)
    _, clean = _step_bits(s, rows, calls[:1])
    _, got = _step_bits(s, rows, calls, unmap=(row, 100))
    for (capacity, live), (hc, sc, err) in zip(calls, got):
        m = capacity if live is None else live
        assert err == cdb.CDB_DEV_UNMAPPED_PAGE
        assert torch.equal(hc[:m], got[0][0][:m]) and torch.equal(sc[:m], got[0][1][:m]), (capacity, live)
    same = (got[0][0] == clean[0][0]).all(1).cpu().numpy()
    assert not same[row] and same[np.arange(66) != row].all()
