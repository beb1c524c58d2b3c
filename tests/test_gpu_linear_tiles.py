"""The matrix-core products (2 to 8 input rows) at the edges of their tiles: K around a block (64), a
round (1,024) and the rounds in flight, N that is odd, below a workgroup's share, and at every
number of tiles per workgroup (1 to 5, and up to four workgroups per compute unit), through qf_linear and
beside a sweep (another decomposition, of one tile a workgroup or two: bitwise the same).

Gate: the bf16 values around the exact result widened by the fp32 accumulation bound of the other
product tests, (K/64 + 32) 2^-24 of the absolute sum.  Infinities and NaN in x, the gains and the
weights: the outputs that are not finite are those of the vector path (one row at a time), and alike."""

import numpy as np
import pytest
import torch

import oracle
import paper_2608_15473_amd as qf
from parity import bf16_neighbours, say
from workloads import make_case

pytestmark = pytest.mark.gpu

CASES = [  # (M, N, K, prologue, residual, split, GLU output)
    (2, 1, 8, None, False, None, False),
    (8, 2, 64, "rms_norm", False, None, True),
    (3, 7, 72, None, True, 3, False),
    (5, 250, 1016, "rms_norm", True, None, False),
    (8, 513, 1024, None, True, 512, False),
    (4, 2050, 1032, "rms_norm", False, None, True),       # 2 tiles, a short second round
    (7, 4602, 2048, "rms_norm", False, 4096, False),      # 3 tiles
    (8, 6400, 3080, None, False, None, True),
    (6, 8001, 1096, "rms_norm", True, None, False),       # 4 tiles
    (2, 10240, 136, None, True, None, False),             # 5 tiles
    (8, 10242, 2120, "rms_norm", False, None, True),      # two workgroups per compute unit: 3 tiles
    (3, 14400, 200, None, False, 7, False),               # 4 tiles
    (8, 20000, 1992, "rms_norm", False, None, False),     # three workgroups: 4 tiles
    (3, 30000, 72, "rms_norm", False, None, False),       # four
    (5, 9001, 2056, "rms_norm", True, None, False),       # one workgroup of 5 tiles, K in 3 rounds
    (7, 9730, 1032, "rms_norm", False, None, True),
    (4, 2600, 2056, None, True, None, False),             # 2 tiles, three rounds in flight: 3,
    (2, 2601, 3080, None, False, 2600, False),            # 4, 5 and 6 rounds
    (8, 2600, 4104, None, False, None, True),
    (3, 2600, 5128, None, False, None, False),
    (6, 1026, 2056, "rms_norm", False, None, True),       # 1 tile, two in flight: 3 rounds
    (8, 264, 9736, None, True, None, False),              # 10 rounds
    (3, 9, (1 << 20) + 8, "rms_norm", True, 4, False),
    (2, 4201, 4168, None, False, None, False),            # beside a sweep: one tile, 526 workgroups
    (2, 4201, 4096, None, False, None, False),            # two tiles, 263
    (3, 1985, 520, "rms_norm", False, 1984, False),       # one tile, all on units of their own
    (5, 1026, 5128, "rms_norm", False, None, True),
]


def _inputs(gpu, M, N, K, pro, res):
    gen = torch.Generator(device=gpu).manual_seed(M * 131 + N * 17 + K)
    x = torch.randn(M, K, generator=gen, device=gpu).to(torch.bfloat16)
    x *= torch.tensor([1.0, 1e-3, 30.0, 1.0, 3.0, 0.5, 1.0, 2.0], device=gpu)[:M, None]
    w = (torch.randn(N, K, generator=gen, device=gpu) / K ** 0.5).to(torch.bfloat16)
    g = (torch.rand(K, generator=gen, device=gpu) + 0.5).to(torch.bfloat16) if pro else None
    r = torch.randn(M, N, generator=gen, device=gpu).to(torch.bfloat16) if res else None
    return x, w, g, r


@pytest.mark.parametrize("M,N,K,pro,res,split,glu", CASES)
def test_tiles_match_the_oracle_and_the_shared_launch(gpu, M, N, K, pro, res, split, glu):
    x, w, g, r = _inputs(gpu, M, N, K, pro, res)
    kw = dict(prologue=pro, gain=g, eps=1e-6, residual=r, split=split, glu_out=glu)
    say(f"[tiles] M={M} N={N} K={K} {pro} residual={res} split={split} glu={glu}")
    got = qf.linear(x, w, **kw)
    case = make_case(2, 4, 2, [300, 17], [2, 1], seed=3, device=gpu)
    beside = qf.attn_decode_split_beside(case.q, case.k_cache, case.v_cache, case.block_table,
                                         case.ctx_lens, case.n_shards, dict(x=x, w=w, **kw),
                                         max_shards=2, scale=case.scale)[2]
    torch.cuda.synchronize()
    got, beside = (torch.cat(t, 1) if split is not None and split < N else t for t in (got, beside))
    assert torch.equal(got.view(torch.int16), beside.view(torch.int16))
    xd, wd = x.double().cpu().numpy(), w.double().cpu().numpy()
    px = oracle.rms_norm(xd, g.double().cpu().numpy(), 1e-6) if pro else xd
    ref, bound = px @ wd.T, np.abs(px) @ np.abs(wd).T
    eps = (K / 64 + 32) * 2.0 ** -24
    if glu:
        gate, up = ref[:, 0::2], ref[:, 1::2]
        ref = oracle.swiglu(gate, up)
        delta = (1.1 * np.abs(up) * eps * bound[:, 0::2]
                 + np.abs(oracle.silu(gate)) * eps * bound[:, 1::2] + 1e-6 * np.abs(ref))
    else:
        rd = r.double().cpu().numpy() if res else 0.0
        ref = ref + rd
        delta = eps * (bound + np.abs(rd))
    lo, _ = bf16_neighbours(ref - delta)
    _, hi = bf16_neighbours(ref + delta)
    out = got.double().cpu().numpy()
    ok = (out >= lo) & (out <= hi)
    assert ok.all(), (np.argwhere(~ok)[:4], out[~ok][:4], ref[~ok][:4])


@pytest.mark.parametrize("pro,glu", [(None, False), ("rms_norm", True)])
def test_rows_too_long_for_the_tiles_are_taken_one_by_one(gpu, pro, glu):
    """K past the tiles' offsets (2^24): by themselves and beside a sweep, each row is bitwise the call
    with that row alone, and the sum that torch gives in fp64."""
    M, N, K = 3, 6, (1 << 24) + 8
    gen = torch.Generator(device=gpu).manual_seed(77)
    x = torch.randn(M, K, generator=gen, device=gpu).to(torch.bfloat16)
    w = (torch.randn(N, K, generator=gen, device=gpu) / 4096).to(torch.bfloat16)
    g = torch.ones(K, device=gpu, dtype=torch.bfloat16) if pro else None
    r = None if glu else torch.randn(M, N, generator=gen, device=gpu).to(torch.bfloat16)
    say(f"[tiles] K={K} {pro} glu={glu}")
    kw = dict(prologue=pro, gain=g, eps=1e-6, glu_out=glu)
    cut = None if glu else 4
    rows = [qf.linear(x[m:m + 1], w, residual=None if glu else r[m:m + 1], split=cut, **kw)
            for m in range(M)]
    got = qf.linear(x, w, residual=r, split=cut, **kw)
    case = make_case(2, 4, 2, [300, 17], [2, 1], seed=3, device=gpu)
    beside = qf.attn_decode_split_beside(case.q, case.k_cache, case.v_cache, case.block_table,
                                         case.ctx_lens, case.n_shards,
                                         dict(x=x, w=w, residual=r, split=cut, **kw), max_shards=2,
                                         scale=case.scale)[2]
    torch.cuda.synchronize()
    got, beside = (torch.cat(t, 1) if cut else t for t in (got, beside))
    want = torch.cat([torch.cat(t, 1) if cut else t for t in rows])
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    assert torch.equal(beside.view(torch.int16), want.view(torch.int16))
    for m in range(M):
        y = (w.double() * x[m].double()).sum(1)
        if pro:
            y = y / torch.sqrt((x[m].double() ** 2).mean() + 1e-6)
        y = y[0::2] * torch.sigmoid(y[0::2]) * y[1::2] if glu else y + r[m].double()
        # sums of 2^24 terms of size 2^-12: (K/64 + 32) 2^-24 of the absolute sum, 2^12 * 0.64, is 41;
        # fp32 sums of random signs stay within a thousandth of it
        torch.testing.assert_close(got[m].double(), y, rtol=2 ** -7, atol=0.05)


@pytest.mark.parametrize("N,K,pro,glu", [(64, 512, None, False), (1024, 3072, None, False),
                                         (6144, 1032, "rms_norm", True), (9000, 1024, "rms_norm", False),
                                         (300, 1000, "swiglu", False)])
def test_a_row_has_the_same_bits_among_any_others(gpu, N, K, pro, glu):
    """2 to 8 rows, in any place (and alone with the SwiGLU input): each row bitwise as among eight."""
    gen = torch.Generator(device=gpu).manual_seed(N + K)
    x = torch.randn(8, 2 * K if pro == "swiglu" else K, generator=gen, device=gpu).to(torch.bfloat16)
    w = (torch.randn(N, K, generator=gen, device=gpu) / K ** 0.5).to(torch.bfloat16)
    g = (torch.rand(K, generator=gen, device=gpu) + 0.5).to(torch.bfloat16) if pro == "rms_norm" else None
    say(f"[tiles] rows among others, N={N} K={K} {pro} glu={glu}")
    full = qf.linear(x, w, pro, g, 1e-6, glu_out=glu).view(torch.int16)
    for m in range(1 if pro == "swiglu" else 2, 8):
        for at in (0, 8 - m):
            got = qf.linear(x[at:at + m], w, pro, g, 1e-6, glu_out=glu).view(torch.int16)
            assert torch.equal(got, full[at:at + m]), (m, at)


@pytest.mark.parametrize("N,K", [(78, k) for k in (1016, 1024, 1032, 1536, 2048, 2560, 10240, 10248, 11776)]
                         + [(2046, 4104), (2050, 4096), (2051, 4104), (2048, 4608), (2050, 11784),
                            (2050, 16384), (2050, 16392)])
@pytest.mark.parametrize("pro,glu", [(None, False), ("rms_norm", False), ("rms_norm", True),
                                     ("swiglu", False)])
def test_one_row_beside_a_sweep_equals_the_call_bitwise(gpu, N, K, pro, glu):
    """The groups of chunks of a single row's K in the shared launch (two or three, whole or not), with
    four output rows a wavefront and with two."""
    if glu and N % 2:
        N += 1
    x, w, g, r = _inputs(gpu, 1, N, K, pro == "rms_norm", not glu)
    if pro == "swiglu":
        x = torch.cat([x, x.flip(1)], 1).contiguous()
    kw = dict(x=x, w=w, prologue=pro, gain=g, residual=r, glu_out=glu)
    case = make_case(2, 4, 2, [300, 17], [2, 1], seed=3, device=gpu)
    say(f"[tiles] one row beside a sweep, N={N} K={K} {pro} glu={glu}")
    got = qf.attn_decode_split_beside(case.q, case.k_cache, case.v_cache, case.block_table,
                                      case.ctx_lens, case.n_shards, kw, max_shards=2,
                                      scale=case.scale)[2]
    want = qf.linear(**kw)
    torch.cuda.synchronize()
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("pro", [None, "rms_norm"])
def test_non_finite_inputs_come_out_as_on_the_vector_path(gpu, pro):
    M, N, K = 6, 40, 1160
    x, w, g, _ = _inputs(gpu, M, N, K, pro, False)
    inf, nan = float("inf"), float("nan")
    x[1, 5], x[2, 1100], x[3, 7] = inf, -inf, nan
    w[3, 9], w[4, 1159], w[5, 0] = inf, -inf, nan
    x[0, 9] = 1.0                     # a factor of few bits against an infinite weight
    w[6, 5] = 0.0                     # 0 times an infinite input
    if g is not None:
        g[700] = inf
        g[701:] = 1.0
    got = qf.linear(x, w, pro, g, 1e-6).float()
    one = torch.cat([qf.linear(x[m:m + 1], w, pro, g, 1e-6) for m in range(M)]).float()
    torch.cuda.synchronize()
    same = torch.isfinite(one)
    assert torch.equal(torch.isnan(got), torch.isnan(one))
    assert torch.equal(got[~same & ~torch.isnan(one)], one[~same & ~torch.isnan(one)])
    torch.testing.assert_close(got[same], one[same], rtol=2 ** -7, atol=1e-4)


@pytest.mark.parametrize("pro,N,K", [(None, 2560, 9728), ("rms_norm", 19456, 2560)])
@pytest.mark.parametrize("bad", [float("nan"), float("inf"), 3e19])   # 3e19: finite, its square is not
def test_a_bad_row_neither_changes_nor_slows_the_others(gpu, pro, N, K, bad):
    """One row of eight that is not finite (a request marked NaN): its outputs are those of the
    vector path, the other rows' bits are the ones they have without it, and the product takes no
    longer than a product of finite rows (1.5 times its time, against 8 to 40 when every NaN
    output is summed again by one thread)."""
    x, w, g, _ = _inputs(gpu, 8, N, K, pro, False)
    y = x.clone()
    y[3] = bad
    say(f"[tiles] a row of {bad}, {pro}, N={N} K={K}")
    good, got = qf.linear(x, w, pro, g, 1e-6), qf.linear(y, w, pro, g, 1e-6)
    one = qf.linear(y[3:4], w, pro, g, 1e-6).float()
    keep = [m for m in range(8) if m != 3]
    assert torch.equal(got[keep].view(torch.int16), good[keep].view(torch.int16))
    row = got[3:4].float()
    assert torch.equal(torch.isnan(row), torch.isnan(one))
    fin = torch.isfinite(one)
    assert torch.equal(row[~fin & ~torch.isnan(one)], one[~fin & ~torch.isnan(one)])
    if pro is None:
        torch.testing.assert_close(row[fin], one[fin], rtol=2 ** -6, atol=1e-3 * abs(3e19))
    else:
        assert torch.equal(row[fin], one[fin])          # a sum of squares of inf: 0 or NaN

    def best(a):
        times = []
        for _ in range(5):
            t = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            t[0].record()
            for _ in range(8):
                qf.linear(a, w, pro, g, 1e-6, out=got)
            t[1].record()
            t[1].synchronize()
            times.append(t[0].elapsed_time(t[1]))
        return min(times)
    best(x)
    base, slow = best(x), best(y)
    assert slow < 1.5 * base, (base, slow)


@pytest.mark.parametrize("M,N,I,K", [(1, 2048, 3072, 1024), (1, 33, 5, 2568), (1, 8, 40, 9736),
                                     (2, 250, 7, 1032), (8, 2048, 3072, 1024), (5, 4095, 6000, 72),
                                     (8, 4096, 9728, 328), (3, 5000, 1, 64)])
def test_pair_equals_the_two_calls_bitwise(gpu, M, N, I, K):
    """A projection and a gated product of the same rows in one launch: every share of rows per
    workgroup, both paths (one row, several), every group of chunks of a row's K."""
    x, wa, ga, _ = _inputs(gpu, M, N, K, "rms_norm", False)
    _, wb, gb, _ = _inputs(gpu, M, 2 * I, K, "rms_norm", False)
    a = dict(x=x, w=wa, prologue="rms_norm", gain=ga, split=(N + 1) // 2)
    b = dict(x=x, w=wb, prologue="rms_norm", gain=gb, glu_out=True)
    say(f"[tiles] pair M={M} N={N} I={I} K={K}")
    (p1, p2), q = qf.linear_pair(a, b)
    (r1, r2), s = qf.linear(**a), qf.linear(**b)
    torch.cuda.synchronize()
    for got, ref in ((p1, r1), (p2, r2), (q, s)):
        assert torch.equal(got.view(torch.int16), ref.view(torch.int16))
    # two products that cannot share a launch
    y, z = qf.linear_pair(b, dict(x=x, w=wa))
    assert torch.equal(y.view(torch.int16), s.view(torch.int16))
    assert torch.equal(z.view(torch.int16), qf.linear(x, wa).view(torch.int16))
