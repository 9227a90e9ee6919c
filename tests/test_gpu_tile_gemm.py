"""GPU: the tile GEMMs at their edges.

Whole prefill chunks against the oracle (tolerances of the prefill tests): row counts
around the 3- and 4-tile row groups and the thresholds where a projection changes
kernel (65, 129, 257 rows), stripe counts that 2 and 3 do not divide, K ranges that
leave waves without a step, with a partial group and with several load groups.

Loop steps and codas bit for bit against smaller calls of the same rows, which run in
the skinny kernel: one and two K parts per wave, 2, 3 and 4 stripes per workgroup, 16
splits, and device row counts that end inside a row tile."""
import numpy as np
import pytest
import torch

import cdbgen
import paper_2608_09444_amd as cdb
from test_gpu_edges import _batch_invariance
from test_gpu_prefill import HD96, ODD, run_prefill
from test_gpu_split_attention import _step_bits

pytestmark = pytest.mark.gpu

# 74 k steps in the down projection: 18 or 19 per wave, two load groups of 8 and a remainder
LONG = cdbgen.shrink(cdbgen.TINY, name="tiny-74", d_ff=1184, r_max=2)


@pytest.mark.parametrize("rows", [64, 65, 97, 128, 129, 161, 256, 257, 289, 512])
@pytest.mark.parametrize("shape", [ODD, HD96, LONG], ids=lambda s: s.name)
def test_chunk_rows(shape, rows):
    w = cdbgen.model_weights(shape)
    prompt = cdbgen.prompt_ids(shape.vocab, 1, rows, seed=90)[0]
    print(f"[gpu] tile GEMM {shape.name}: {rows} rows", flush=True)
    err = run_prefill(shape, w, prompt, [rows])
    print(f"[gpu]   {err}", flush=True)


@pytest.mark.parametrize("rows,alone", [(129, 64), (200, 128), (256, 33)])
def test_loop_step_rows_keep_their_bits_above_128(rows, alone):
    """The tile kernel's two-part passes against the skinny kernel's 8 waves, the same rows."""
    s = cdbgen.shrink(cdbgen.OURO, name="ouro-1-layer", vocab=64, n_core=1)
    r = cdbgen.decode_snapshot(rows, cdbgen.OURO_DEPTHS, s.r_max, 5, 60, stream=93)
    print(f"[gpu] {rows} rows vs their first {alone}", flush=True)
    _batch_invariance(s, cdbgen.model_weights(s), r, alone)


@pytest.mark.parametrize("rows,alone", [(129, 64), (256, 128)])
def test_many_splits_keep_their_bits_above_128(rows, alone):
    """A long reduction onto few columns takes 16 splits (more than the tile kernel's own choice ever is)."""
    s = cdbgen.shrink(cdbgen.TINY, name="512-16384", d=512, n_heads=8, d_ff=16384, vocab=64, n_prelude=0, n_core=1,
                      n_coda=0)
    r = cdbgen.decode_snapshot(rows, cdbgen.OURO_DEPTHS, s.r_max, 5, 60, stream=94)
    print(f"[gpu] 16 splits: {rows} rows vs their first {alone}", flush=True)
    _batch_invariance(s, cdbgen.model_weights(s), r, alone)


def _same_as_first(calls, h0, got):
    h, score, _ = got[0]
    for (capacity, live), (hc, sc, err) in zip(calls, got):
        m = capacity if live is None else live
        assert err == 0
        assert torch.equal(hc[:m], h[:m]) and torch.equal(sc[:m], score[:m]), (capacity, live)
        assert torch.equal(hc[m:], h0[m:]), (capacity, live)


def test_long_reductions_and_device_counts_keep_their_bits():
    """Huginn widths (165 stripes, an adapter and 3 K splits), where the tile kernel runs from 65 rows on and takes 4
    stripes and 3 row tiles at 129-192 rows, 3 stripes and 4 row tiles above, against 50 rows in the skinny kernel."""
    s = cdbgen.shrink(cdbgen.HUGINN, name="huginn-1-layer", d_ff=2560, vocab=64, n_prelude=0, n_core=1, n_coda=0)
    r = cdbgen.decode_snapshot(256, cdbgen.WORKLOADS[3].depth, s.r_max, 5, 60, stream=95)
    calls = [(256, None), (50, None), (65, None), (97, None), (140, None), (192, None), (100, 70), (100, 33), (140, 129),
             (192, 50), (256, 193), (256, 0)]
    print("[gpu] Huginn widths", flush=True)
    _same_as_first(calls, *_step_bits(s, r, calls))


def test_two_part_tiles_keep_their_bits_under_a_device_count():
    s = cdbgen.shrink(cdbgen.OURO, name="ouro-1-layer", vocab=64, n_core=1)
    r = cdbgen.decode_snapshot(256, cdbgen.OURO_DEPTHS, s.r_max, 5, 60, stream=96)
    calls = [(256, None), (128, None), (64, None), (129, 129), (140, 100), (200, 129), (200, 31), (256, 193), (256, 1)]
    print("[gpu] Ouro widths", flush=True)
    _same_as_first(calls, *_step_bits(s, r, calls))


def test_lm_head_of_four_stripes_keeps_its_bits():
    """800 stripes at 129-192 rows take 4 per workgroup, at 193-256 rows 3 with 4 row tiles; against 64 rows."""
    s = cdbgen.shrink(cdbgen.TINY, name="512-lm", d=512, n_heads=8, d_ff=96, vocab=25600, n_prelude=0, n_core=1, n_coda=1)
    n = 256
    ar = np.arange(n, dtype=np.int32)
    pos = (ar % 16).astype(np.int32)
    kv = cdb.PagedKV(s, n, 1, 0, 1, n, fill="random")
    g = torch.Generator(device="cuda")
    g.manual_seed(97)
    kv.coda.normal_(0.0, 1.0, generator=g)
    pt = np.full((n, s.r_max + 2, 1), -1, np.int32)
    pt[:, s.r_max + 1, 0] = ar
    kv.page_table.copy_(torch.from_numpy(pt))
    coda0 = kv.coda.clone()
    state = cdb.State(s, n)
    state.h.normal_(0.0, 1.0, generator=g)
    gm = cdb.DeviceModel(s, cdbgen.model_weights(s))
    ws = cdb.Workspace(gm.desc, n)
    first = None
    for capacity, live in ((64, None), (129, None), (192, None), (193, None), (256, None), (140, 61), (256, 33)):
        print(f"[gpu] LM head: {capacity} rows, {live} live", flush=True)
        kv.coda.copy_(coda0)
        count = None if live is None else torch.tensor([live], dtype=torch.int32, device="cuda")
        rows = cdb.Rows(ar[:capacity], ar[:capacity], pos[:capacity], d_n_rows=count)
        logits = torch.full((capacity, s.vocab), -7.0, dtype=torch.float32, device="cuda")
        ids = torch.full((capacity,), -7, dtype=torch.int32, device="cuda")
        cdb.cdb_boundary_coda(gm.model, kv.c, state.c, rows.c, logits, ids, ws.buf)
        torch.cuda.synchronize()
        assert cdb.cdb_read_device_error(ws.buf) == 0
        m = min(capacity if live is None else live, 64)
        if first is None:
            first = (logits, ids)
        assert torch.equal(logits[:m], first[0][:m]) and torch.equal(ids[:m], first[1][:m]), (capacity, live)
        if live is not None:
            assert bool((logits[live:] == -7.0).all()) and bool((ids[live:] == -7).all())


@pytest.mark.parametrize("vocab", [1024, 8192])
def test_logits_may_start_at_any_float(vocab):
    """Prefill and coda into logits that are aligned to 4 bytes only: the bits of a 256-byte aligned array."""
    s = cdbgen.shrink(cdbgen.TINY, name=f"tiny-v{vocab}", vocab=vocab, n_prelude=0, n_core=1, n_coda=0, r_max=1)
    gm = cdb.DeviceModel(s, cdbgen.model_weights(s))
    n = 330
    pages = cdbgen.pages_for(n)
    kv = cdb.PagedKV(s, 1, pages, 0, pages, 0, fill="random")
    kv.page_table.copy_(torch.arange(pages, dtype=torch.int32).expand(1, s.r_max + 2, pages))
    ws = cdb.Workspace(gm.desc, n)
    state = cdb.State(s, n)
    state.h.normal_(0.0, 1.0)
    tok = torch.as_tensor(cdbgen.prompt_ids(vocab, 1, n, seed=98)[0], dtype=torch.int32, device="cuda")
    ar = np.arange(n, dtype=np.int32)
    for call, rows in (("prefill", 20), ("prefill", 129), ("prefill", 200), ("prefill", n), ("coda", 20), ("coda", 140),
                       ("coda", 256)):
        print(f"[gpu] {call} of {rows} rows, vocabulary {vocab}, logits at every float of 16 bytes", flush=True)
        want = None
        for first in range(4):
            buf = torch.full((rows * vocab + 8,), -7.0, dtype=torch.float32, device="cuda")
            logits = buf[first:first + rows * vocab]
            ids = torch.empty(rows, dtype=torch.int32, device="cuda")
            if call == "prefill":
                cdb.cdb_prefill(gm.model, kv.c, 0, 0, tok[:rows], logits, ids, ws.buf)
            else:
                r = cdb.Rows(ar[:rows], np.zeros(rows, np.int32), ar[:rows])
                cdb.cdb_boundary_coda(gm.model, kv.c, state.c, r.c, logits, ids, ws.buf)
            torch.cuda.synchronize()
            assert cdb.cdb_read_device_error(ws.buf) == 0
            want = want or (logits, ids)
            assert torch.equal(logits, want[0]) and torch.equal(ids, want[1]), (call, rows, first)
            assert bool((buf[:first] == -7.0).all()) and bool((buf[first + rows * vocab:] == -7.0).all())
