"""The short-shard sweep's deal of units to XCDs (items of all KV heads of a (request, shard, chunk),
or of single units, in rotated rows of 8) at the sizes where it can lose or repeat a unit: item
counts around multiples of 8 and around the rule between the two item sizes, KV head counts that
are no power of two.  Every unit's output is checked against the fp64 oracle at the parity gates,
over buffers that hold NaN before the call, and the one-launch decode (whose count of finished units
would hang the merge or run it early if one were lost) against the two calls."""

import numpy as np
import pytest
import torch

import paper_2608_15473_amd as qf
from parity import check, oracle_ref, run_gpu, say
from workloads import make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,shards,hkv,G", [
    (1, 1, 1, 1), (1, 7, 3, 2), (3, 3, 2, 4), (9, 7, 3, 1), (8, 8, 5, 1), (5, 13, 3, 2), (13, 9, 7, 2),
    (72, 1, 11, 1),
])
def test_every_unit_is_swept_once(gpu, batch, shards, hkv, G):
    rng = np.random.default_rng(1000 * batch + shards)
    ctx = rng.integers(0, 40 * shards, size=batch)
    ctx[0] = 40 * shards
    case = make_case(batch, G * hkv, hkv, ctx, np.minimum(shards, 1 + ctx // 16), seed=900 + batch,
                     max_shards=shards, device=gpu)
    say(f"[deal] batch {batch}, {shards} shards, {hkv} KV heads, G {G}")
    got = run_gpu(case)
    check(case, got, oracle_ref(case), label="deal")
    out, lse = qf.attn_decode(case.q, case.k_cache, case.v_cache, case.block_table, case.ctx_lens,
                              case.n_shards, max_shards=shards, scale=case.scale)
    torch.cuda.synchronize()
    np.testing.assert_allclose(lse.cpu().numpy(), got["lse"], rtol=1e-6, atol=1e-6)
    if qf.split_chunks(qf.make_desc(case.q, case.k_cache, case.block_table, shards, case.scale)) == 1:
        assert np.array_equal(out.view(torch.int16).cpu().numpy(), got["out_bits"])


@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("max_pages", [48, 128])   # the deep short-shard buffers, the long-shard ones
def test_every_number_of_pages_per_wavefront(gpu, G, max_pages):
    """One shard per request of 1 to 48 pages (0 to 12 per wavefront), whole and partial: the page
    buffers' first group, loop and end at every remainder.  Sampled heads, at the parity gates."""
    pages = np.arange(1, 49)
    ctx = 16 * pages - (pages * 7) % 16
    hkv = 24                                           # enough units for unchunked shards
    case = make_case(48, G * hkv, hkv, ctx, 1, seed=950 + G, max_pages=max_pages, device=gpu)
    desc = qf.make_desc(case.q, case.k_cache, case.block_table, 1, case.scale)
    assert qf.split_chunks(desc) == 1
    say(f"[deal] 1 to 48 pages, G {G}, capacity {max_pages}")
    pairs = [(b, (b * 5 + i * (G * hkv // 4 + 1)) % (G * hkv)) for b in range(48) for i in range(4)]
    got = run_gpu(case)
    check(case, got, oracle_ref(case, pairs), pairs, label="pages")
