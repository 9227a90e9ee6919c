"""GPU: the prefill's tile GEMMs at their edges, through whole chunks against the
oracle (tolerances of the prefill tests): row counts around the 3- and 4-tile row
groups and the thresholds where a projection changes kernel (65, 129, 257 rows),
stripe counts that 2, 3 and 4 do not divide, K ranges that leave waves without a
step, with a partial group and with several load groups."""
import pytest

import cdbgen
from test_gpu_edges import _batch_invariance
from test_gpu_prefill import HD96, ODD, run_prefill

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
