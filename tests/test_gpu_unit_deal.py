"""The short-shard sweep's deal of units to XCDs (items of all KV heads of some consecutive (shard,
chunk) slots, or of single units, in rotated rows of 8) at the sizes where it can lose or repeat a
unit: item counts around multiples of 8, items of one slot and of several with a partial last one, on
both sides of the rules between the item sizes (whose constants are read from the sources, so that
a moved threshold moves no case to another item size unseen), KV head counts that are no power of two.
Every unit's output is checked against the fp64 oracle at the parity gates, over buffers that hold
NaN before the call, and the one-launch decode (whose count of finished units would hang the merge or
run it early if one were lost) against the two calls.  Then every number of pages of a wavefront, for
each depth of the page buffers."""

import os
import re

import numpy as np
import pytest
import torch

import paper_2608_15473_amd as qf
from parity import check, oracle_ref, run_gpu, say
from workloads import make_case

pytestmark = pytest.mark.gpu

CONST = dict(re.findall(r"constexpr int (k\w+) = (\d+);", open(os.path.join(
    os.path.dirname(qf.__file__), "csrc", "qf_internal.h")).read()))
MANY, FEW, ITEM, DEEP_MANY = (int(CONST[k]) for k in ("kDealManyUnits", "kDealFewUnits",
                                                      "kDealItemUnits", "kDeepManyUnits"))


def _units_per_item(batch, slots, hkv):
    """The rule between the item sizes, restated."""
    n, units, k = batch * slots, batch * slots * hkv, -(-slots // 8)
    load = lambda k: -(-(-(-n // k)) // 8) * k
    if batch == 1:
        good = -(-slots // k) >= 7 if units <= FEW else load(k) * 64 <= n * 9
        return k * hkv if good else -(-units // 8)
    if units < MANY:
        k = -(-ITEM // hkv)
    if units <= FEW and -(-n // k) >= 8:
        return k * hkv
    least = min(load(i) for i in range(1, k + 1))
    if least * 64 > n * 9:
        return 1
    return max(i for i in range(1, k + 1) if load(i) * 32 <= least * 33) * hkv


@pytest.mark.parametrize("batch,shards,hkv,G,item", [
    (1, 1, 1, 1, 1), (1, 7, 3, 2, 3), (3, 3, 2, 4, 1), (9, 7, 3, 1, 9), (8, 8, 5, 1, 10), (5, 13, 3, 2, 9),
    (13, 9, 7, 2, 7), (72, 1, 11, 1, 11),
    (1, 65, 3, 1, 27), (1, 26, 2, 1, 8),      # few units of one request: an eighth of the slots, the last item short
    (1, 4, 24, 1, 12), (1, 9, 5, 2, 6),       # or of the units, slots cut
    (1, 300, 8, 2, 304), (1, 43, 7, 4, 42),   # more: of the slots where even,
    (1, 42, 7, 1, 37),                        # of the units where not
    (7, 13, 1, 2, 8), (3, 27, 2, 1, 8),       # few units of several requests: of eight, the last item short
    (10, 20, 5, 1, 5), (24, 17, 1, 2, 4),     # more: fewer slots where eight are less even
    (23, 29, 7, 1, 28),                       # many units of several requests, 167 items
])
def test_every_unit_is_swept_once(gpu, batch, shards, hkv, G, item):
    rng = np.random.default_rng(1000 * batch + shards)
    ctx = rng.integers(0, 40 * shards, size=batch)
    ctx[0] = 40 * shards
    case = make_case(batch, G * hkv, hkv, ctx, np.minimum(shards, 1 + ctx // 16), seed=900 + batch,
                     max_shards=shards, device=gpu)
    chunks = qf.split_chunks(qf.make_desc(case.q, case.k_cache, case.block_table, shards, case.scale))
    assert _units_per_item(batch, shards * chunks, hkv) == item
    say(f"[deal] batch {batch}, {shards} shards, {hkv} KV heads, G {G}, items of {item} units")
    got = run_gpu(case)
    check(case, got, oracle_ref(case), label="deal")
    out, lse = qf.attn_decode(case.q, case.k_cache, case.v_cache, case.block_table, case.ctx_lens,
                              case.n_shards, max_shards=shards, scale=case.scale)
    torch.cuda.synchronize()
    np.testing.assert_allclose(lse.cpu().numpy(), got["lse"], rtol=1e-6, atol=1e-6)
    if chunks == 1 and shards <= 64:
        assert np.array_equal(out.view(torch.int16).cpu().numpy(), got["out_bits"])


@pytest.mark.parametrize("G,max_pages,repeat", [
    (1, 48, 1), (2, 48, 1),      # three page buffers (few units of short shards at G <= 2)
    (1, 48, 4), (2, 48, 4),      # four (many units)
    (4, 48, 1), (8, 48, 1),      # three at G = 4, two at G = 8
    (1, 128, 1), (2, 128, 1), (4, 128, 1), (8, 128, 1),      # long shards: two
])
def test_every_number_of_pages_per_wavefront(gpu, G, max_pages, repeat):
    """One shard per request of 1 to 48 pages (0 to 12 per wavefront), whole and partial: the page
    buffers' first group, loop and end at every remainder, for each depth of the buffers.  Sampled
    heads, at the parity gates."""
    pages = np.tile(np.arange(1, 49), repeat)
    ctx = 16 * pages - (pages * 7 + np.arange(len(pages)) // 48 * 5) % 16
    hkv = 24                                           # enough units for unchunked shards
    units = 48 * repeat * hkv
    assert (units >= DEEP_MANY) == (repeat == 4) and units // repeat < DEEP_MANY
    case = make_case(48 * repeat, G * hkv, hkv, ctx, 1, seed=950 + G, max_pages=max_pages, device=gpu)
    desc = qf.make_desc(case.q, case.k_cache, case.block_table, 1, case.scale)
    assert qf.split_chunks(desc) == 1
    say(f"[deal] 1 to 48 pages, G {G}, capacity {max_pages}, {units} units")
    rows = [b + 48 * (b % repeat) for b in range(48)]   # of each page count, one request
    pairs = [(b, (b * 5 + i * (G * hkv // 4 + 1)) % (G * hkv)) for b in rows for i in range(4)]
    got = run_gpu(case)
    check(case, got, oracle_ref(case, pairs), pairs, label="pages")


@pytest.mark.slow
def test_as_many_units_as_a_launch_takes(gpu):
    """2^24 - 8 units of a short-shard sweep (a launch takes 2^24 - 1 workgroups of 256 threads): no
    workgroup more than units.  Three requests hold positions; bitwise those three alone."""
    B, S, H = 6223, 337, 8
    live = [0, 3000, B - 1]
    few = make_case(3, H, H, [5392, 17, 2048], S, seed=990, max_pages=S, device=gpu)
    table = torch.full((B, S), -1, dtype=torch.int32, device=gpu)
    ctx = torch.zeros(B, dtype=torch.int32, device=gpu)
    q = torch.zeros(B, H, 128, dtype=torch.bfloat16, device=gpu)
    table[live], ctx[live], q[live] = few.block_table, few.ctx_lens, few.q
    say(f"[deal] {B * S * H} units")
    po, pl = qf.attn_decode_split(q, few.k_cache, few.v_cache, table, ctx, S, max_shards=S,
                                  scale=few.scale)
    ref_o, ref_l = qf.attn_decode_split(few.q, few.k_cache, few.v_cache, few.block_table,
                                        few.ctx_lens, few.n_shards, max_shards=S, scale=few.scale)
    torch.cuda.synchronize()
    assert torch.equal(pl[live].view(torch.int32), ref_l.view(torch.int32))
    some = torch.isfinite(ref_l)
    assert torch.equal(po[live][some].view(torch.int32), ref_o[some].view(torch.int32))
    pl[live] = float("-inf")
    assert bool((pl == float("-inf")).all())
    del po, ref_o
    torch.cuda.empty_cache()
