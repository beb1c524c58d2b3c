"""The launches of a block's attention tail at one request (qf_linear_beside_merge,
qf_linear_attn_current) against the calls they stand for, and the stack at one request.

* the product beside the merge: bitwise qf_linear, and qf_attn_combine's values before its rounding;
* the fold: attn within one bf16 step, and lse within 1e-6, of qf_attn_combine_current on the same
  partials (the score of the current token is summed in another order: 128 fp32 terms); exactly the
  current value for an empty cache; the appended token, ctx_lens and status bitwise those of
  qf_kv_append; the product bitwise qf_linear of the attention written;
* the stack's three modes bitwise equal, eagerly and replayed."""

import numpy as np
import pytest
import torch

import paper_2608_15473_amd as qf
from parity import say
from test_gpu_stage import SHAPE, _build, _restore, _same_state, _state
from workloads import BlockShape, make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,ctx,shards,N", [
    (1, 1, 17, 1, 4), (2, 1, 0, 2, 9), (4, 2, 300, 3, 250), (16, 8, 4608, 24, 1024),
    (40, 5, 1000, 64, 2560), (32, 8, 2031, 128, 33), (64, 8, 700, 300, 1000),
])
def test_tail_launches_equal_the_calls_they_stand_for(gpu, hq, hkv, ctx, shards, N):
    case = make_case(1, hq, hkv, [ctx + 1], [shards], seed=70 + hq, max_shards=shards, device=gpu)
    case.ctx_lens -= 1
    gen = torch.Generator(device=gpu).manual_seed(hq * 7 + ctx)

    def draw(*shape):
        return torch.randn(*shape, generator=gen, device=gpu).to(torch.bfloat16)

    H, D = 512, 128
    z, g1 = draw(1, H), (torch.rand(H, generator=gen, device=gpu) + 0.5).to(torch.bfloat16)
    w_kv, w_o, res = draw(2 * hkv * D, H) * 0.05, draw(N, hq * D) * 0.05, draw(1, N)
    say(f"[one] hq={hq} hkv={hkv} ctx={ctx} shards={shards} N={N}")
    po, pl = qf.attn_decode_split(case.q, case.k_cache, case.v_cache, case.block_table,
                                  case.ctx_lens, case.n_shards, max_shards=shards,
                                  scale=case.scale)
    mo = torch.full((1, hq, D), float("nan"), device=gpu)
    ml = torch.full((1, hq), float("nan"), device=gpu)
    kv = dict(x=z, w=w_kv, prologue="rms_norm", gain=g1, split=hkv * D)
    k, v = qf.linear_beside_merge(kv, po, pl, mo, ml)
    for got, ref in zip((k, v), qf.linear(**kv)):
        assert torch.equal(got.view(torch.int16), ref.view(torch.int16))
    out, lse = qf.attn_combine(po, pl)
    torch.testing.assert_close(ml, lse, rtol=1e-6, atol=1e-6)
    if ctx:
        torch.testing.assert_close(mo.to(torch.bfloat16).float(), out.float(), rtol=2 ** -7, atol=0)

    k, v = k.view(1, hkv, D), v.view(1, hkv, D)
    ref_attn, ref_lse = qf.attn_combine_current(po, pl, case.q, k, v, scale=case.scale)
    caches = [(t.clone()) for t in (case.k_cache, case.v_cache, case.ctx_lens)]
    qf.kv_append(*caches[:2], case.block_table, caches[2], k, v)
    attn = torch.full((1, hq, D), float("nan"), device=gpu).to(torch.bfloat16)
    lse = torch.full((1, hq), float("nan"), device=gpu)
    status = torch.zeros(1, dtype=torch.int32, device=gpu)
    y = qf.linear_attn_current(mo, ml, case.q, k, v, attn, lse, case.k_cache, case.v_cache,
                               case.block_table, case.ctx_lens, w_o, scale=case.scale,
                               residual=res, status=status)
    torch.cuda.synchronize()
    torch.testing.assert_close(attn.float(), ref_attn.float(), rtol=2 ** -7,
                               atol=1e-5 * float(ref_attn.float().abs().max()))
    torch.testing.assert_close(lse, ref_lse, rtol=1e-6, atol=1e-6)
    if ctx == 0:
        assert torch.equal(attn[0], v[0].repeat_interleave(hq // hkv, 0))
    assert torch.equal(case.k_cache.view(torch.int16), caches[0].view(torch.int16))
    assert torch.equal(case.v_cache.view(torch.int16), caches[1].view(torch.int16))
    assert case.ctx_lens.tolist() == [ctx + 1] and int(status) == 0
    want = qf.linear(attn.view(1, -1), w_o, residual=res)
    assert torch.equal(y.view(torch.int16), want.view(torch.int16))


def test_a_full_cache_and_two_requests_are_refused(gpu):
    """No room for the token: the cache and its length stay, status is set; two requests: refused."""
    case = make_case(1, 4, 2, [32], [1], seed=5, device=gpu)
    mo, ml = torch.zeros(1, 4, 128, device=gpu), torch.zeros(1, 4, device=gpu)
    k = torch.ones(1, 2, 128, device=gpu).to(torch.bfloat16)
    attn, w = torch.empty_like(case.q), torch.zeros(8, 512, device=gpu).to(torch.bfloat16)
    status = torch.zeros(1, dtype=torch.int32, device=gpu)
    before = case.k_cache.clone()
    qf.linear_attn_current(mo, ml, case.q, k, k, attn, None, case.k_cache, case.v_cache,
                           case.block_table, case.ctx_lens, w, scale=case.scale, status=status)
    torch.cuda.synchronize()
    assert int(status) == 1 and case.ctx_lens.tolist() == [32]
    assert torch.equal(case.k_cache.view(torch.int16), before.view(torch.int16))
    two = make_case(2, 4, 2, [20, 20], [1, 1], seed=6, device=gpu)
    with pytest.raises(qf.QFError) as e:
        qf.linear_attn_current(torch.zeros(2, 4, 128, device=gpu), torch.zeros(2, 4, device=gpu),
                               two.q, k.repeat(2, 1, 1), k.repeat(2, 1, 1), torch.empty_like(two.q),
                               None, two.k_cache, two.v_cache, two.block_table, two.ctx_lens, w)
    assert e.value.code == qf.QF_EUNSUPPORTED


MANY = BlockShape("many heads", hidden=256, inter=512, n_q_heads=72, n_kv_heads=9, layers=3)


@pytest.mark.parametrize("ctx,shards,shape", [(300, 3, SHAPE), (0, 1, SHAPE), (2, 2, SHAPE), (77, 2, MANY)])
def test_stack_of_one_request_in_all_modes(gpu, ctx, shards, shape):
    stack, u = _build(gpu, seed=810, ctx=np.array([ctx]), shards=[shards], shape=shape)
    assert stack.short_tail == (shape is SHAPE)
    saved = _state(stack)
    ys, states = {}, {}
    for mode in ("serial", "streams", "fused"):
        say(f"[one] stack, {ctx} positions, mode {mode}")
        _restore(stack, saved)
        ys[mode] = [stack.step(u, mode=mode).clone() for _ in range(2)]
        torch.cuda.synchronize()
        states[mode] = _state(stack)
    for mode in ("streams", "fused"):
        assert all(torch.equal(a, b) for a, b in zip(ys["serial"], ys[mode])), mode
        assert _same_state(states["serial"], states[mode]), mode
    assert int(stack.status.item()) == 0 and stack.caches[0].ctx_lens.tolist() == [ctx + 2]
    # the last block, from the stack's own tensors
    w = stack.layers[-1]
    y = qf.linear(stack.attn.view(1, -1), w["w_o"], residual=stack.z)
    assert torch.equal(y.view(torch.int16), ys["fused"][-1].view(torch.int16))
    graph, out = stack.capture(u)
    for r in range(3):
        _restore(stack, saved)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ys["serial"][0]), r
        stack.step(u, mode="serial")
        torch.cuda.synchronize()
    assert shape.layers == len(stack.layers)
