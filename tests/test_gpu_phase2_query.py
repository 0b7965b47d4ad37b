"""Parity of pulsar_phase2_query with oracle.attention.query_attention.

New tokens attend, without a mask, to the retained shards and to the
generation shard's appended rows up to themselves (Algorithm 1, Phase 2).
Acceptance as for the other attention outputs: O max-abs 1e-2 and relative
L2 1e-2, LSE max-abs 1e-3.
"""
import math

import numpy as np
import pytest
import torch

import paper_2607_20457_amd as P
from oracle import attention as oatt
from paper_2607_20457_amd import workload
from tests._helpers import check_attention, f64, to_dev_bf16

pytestmark = pytest.mark.gpu


def _run_and_check(q, kg, vg, G, k=None, v=None, what=""):
    d = q.shape[-1]
    scale = 1.0 / math.sqrt(d)
    print(f"phase2_query parity: {what}", flush=True)
    o, lse = P.phase2_query(to_dev_bf16(q), to_dev_bf16(kg), to_dev_bf16(vg), G,
                            None if k is None else to_dev_bf16(k),
                            None if v is None else to_dev_bf16(v))
    Hkv = kg.shape[1]
    Ks = f64(k) if k is not None else np.zeros((0, 0, Hkv, d))
    Vs = f64(v) if v is not None else np.zeros((0, 0, Hkv, d))
    o_ref, lse_ref = oatt.query_attention(f64(q), Ks, Vs, f64(kg), f64(vg), G, scale)
    check_attention(o.cpu().numpy(), lse.cpu().numpy(), o_ref, lse_ref, what)


def test_query_encoding_over_128k_shards():
    # 64 query tokens over the 16 retained shards of 8192 keys (the 128K
    # workload's K/V), then their own rows causally
    cfg = workload.CONFIGS["llama8b_128k"]
    _, k, v = workload.make_qkv(cfg, batch=1)
    Ks = np.ascontiguousarray(k[0].reshape(16, 8192, cfg.Hkv, cfg.d))
    Vs = np.ascontiguousarray(v[0].reshape(16, 8192, cfg.Hkv, cfg.d))
    q = workload.bf16_normal(501, (64, cfg.Hq, cfg.d))
    kg = workload.bf16_normal(502, (64, cfg.Hkv, cfg.d))
    vg = workload.bf16_normal(503, (64, cfg.Hkv, cfg.d))
    _run_and_check(q, kg, vg, 0, Ks, Vs, "query encoding 16 x 8192")


@pytest.mark.parametrize("G", [1, 70, 300])
def test_decode_step(G):
    q = workload.bf16_normal(600 + G, (1, 32, 128))
    kg = workload.bf16_normal(601 + G, (G + 1, 8, 128))
    vg = workload.bf16_normal(602 + G, (G + 1, 8, 128))
    k = workload.bf16_normal(603, (4, 512, 8, 128))
    v = workload.bf16_normal(604, (4, 512, 8, 128))
    _run_and_check(q, kg, vg, G, k, v, f"decode G={G}")


@pytest.mark.parametrize("Hq,Hkv,d,Tq,G,ns,S", [
    (32, 8, 128, 40, 5, 0, 0),       # generation shard only, ragged
    (32, 8, 128, 33, 0, 3, 0),       # empty retained shards
    (4, 1, 64, 100, 17, 2, 300),     # the small layer shape, d 64
    (8, 8, 128, 65, 3, 5, 129),      # one query head per KV head
    (16, 8, 64, 31, 0, 6, 77),       # two query heads per KV head
    (32, 8, 128, 40, 4100, 1, 256),  # generation shard over 4096 rows: attention kernel
    (64, 1, 64, 3, 10, 1, 100),      # 64 heads per KV head: no 32-row tile, attention kernel
    (32, 8, 128, 130, 20, 1, 64),    # 520 query rows per KV head: attention kernel, G > 0
    (64, 8, 64, 13, 7, 2, 90),       # 8 heads per KV head: tiles of 4 tokens, the last of 1
    (32, 1, 64, 5, 3, 1, 50),        # 32 heads per KV head: one token per tile
])
def test_shapes(Hq, Hkv, d, Tq, G, ns, S):
    seed = Hq * 7 + Tq + G
    q = workload.bf16_normal(seed, (Tq, Hq, d))
    kg = workload.bf16_normal(seed + 1, (G + Tq, Hkv, d))
    vg = workload.bf16_normal(seed + 2, (G + Tq, Hkv, d))
    k = workload.bf16_normal(seed + 3, (ns, S, Hkv, d)) if ns else None
    v = workload.bf16_normal(seed + 4, (ns, S, Hkv, d)) if ns else None
    _run_and_check(q, kg, vg, G, k, v, f"Hq={Hq} Hkv={Hkv} d={d} Tq={Tq} G={G} shards={ns}x{S}")


def test_peaked_queries():
    # queries scaled x8: the weights concentrate and |O| is of order 1
    q = workload.bf16_normal(700, (16, 32, 128), scale=8.0)
    kg = workload.bf16_normal(701, (16 + 9, 8, 128))
    vg = workload.bf16_normal(702, (16 + 9, 8, 128))
    k = workload.bf16_normal(703, (8, 1024, 8, 128))
    v = workload.bf16_normal(704, (8, 1024, 8, 128))
    _run_and_check(q, kg, vg, 9, k, v, "peaked")


@pytest.mark.parametrize("Hq,Hkv,d,Tq,G,ns,S", [
    (32, 8, 128, 8, 5, 3, 700),      # 32 packed rows: the decode kernel, causal new rows
    (8, 8, 128, 32, 0, 0, 0),        # one head per KV head, new tokens only
    (16, 8, 64, 16, 600, 2, 300),    # generation shard in three key ranges
    (32, 8, 128, 3, 2000, 4, 512),   # eight generation ranges, the last holding the new rows
    (4, 1, 64, 7, 0, 1, 100),        # one KV head
    (32, 1, 128, 1, 40, 2, 333),     # 32 heads per KV head, one token: a full tile
    (32, 8, 128, 1, 0, 0, 0),        # one token, nothing before it: its own row only
])
def test_few_rows_one_launch(Hq, Hkv, d, Tq, G, ns, S):
    # Tq * Hq / Hkv <= 32: shards and generation shard in one decode launch,
    # token t limited to generation rows up to G + t
    seed = 900 + Hq + Tq + G
    q = workload.bf16_normal(seed, (Tq, Hq, d))
    kg = workload.bf16_normal(seed + 1, (G + Tq, Hkv, d))
    vg = workload.bf16_normal(seed + 2, (G + Tq, Hkv, d))
    k = workload.bf16_normal(seed + 3, (ns, S, Hkv, d)) if ns else None
    v = workload.bf16_normal(seed + 4, (ns, S, Hkv, d)) if ns else None
    _run_and_check(q, kg, vg, G, k, v, f"few rows Hq={Hq} Hkv={Hkv} d={d} Tq={Tq} G={G} "
                   f"shards={ns}x{S}")


@pytest.mark.parametrize("Hq,Hkv,d,Tq,G,ns,S", [
    (32, 8, 128, 9, 0, 2, 129),      # two row tiles, the second of 4 rows; a step past one range
    (32, 8, 128, 16, 0, 1, 31),      # two full tiles, less than one step
    (32, 8, 128, 17, 40, 3, 700),    # three tiles: the last tile group half empty
    (32, 8, 128, 32, 0, 4, 1024),    # four full tiles, whole ranges
    (24, 2, 128, 8, 3, 2, 200),      # 12 heads per KV head: tiles of 24 live rows
    (64, 2, 128, 3, 500, 1, 90),     # 32 heads per KV head: one token per tile
    (32, 8, 128, 20, 300, 32, 40),   # a full chip: the generation rows join the shards' ranges
    (32, 8, 128, 20, 9000, 1, 5000), # long generation shard, ranges of its own
    (16, 16, 64, 33, 0, 2, 127),     # d 64: two tiles, the second of one row
    (16, 16, 64, 64, 7, 16, 65),     # d 64: two full tiles, generation rows joined
    (16, 4, 64, 44, 10, 2, 640),     # d 64: six tiles, three per wave
    (16, 4, 64, 37, 1000, 0, 0),     # d 64: five tiles, generation shard only
])
def test_packed_rows(Hq, Hkv, d, Tq, G, ns, S):
    # a few dozen tokens: 32-row tiles of packed (token, head) rows
    seed = 1300 + Hq + Tq + G
    q = workload.bf16_normal(seed, (Tq, Hq, d))
    kg = workload.bf16_normal(seed + 1, (G + Tq, Hkv, d))
    vg = workload.bf16_normal(seed + 2, (G + Tq, Hkv, d))
    k = workload.bf16_normal(seed + 3, (ns, S, Hkv, d)) if ns else None
    v = workload.bf16_normal(seed + 4, (ns, S, Hkv, d)) if ns else None
    _run_and_check(q, kg, vg, G, k, v, f"packed Hq={Hq} Hkv={Hkv} d={d} Tq={Tq} G={G} "
                   f"shards={ns}x{S}")


def test_packed_far_larger_later_score():
    # one key far above every row's first scores (a weight sum past 2^88): the
    # workgroup that holds it repeats its range with a raised reference
    Tq, Hq, Hkv, d, S = 20, 8, 2, 128, 700
    q = workload.bf16_bits_to_f32(workload.bf16_normal(1401, (Tq, Hq, d))) + 1.0
    kf = workload.bf16_bits_to_f32(workload.bf16_normal(1402, (2, S, Hkv, d)))
    kf[1, 400] = 8.0
    qb, kb = workload.f32_to_bf16_bits(q), workload.f32_to_bf16_bits(kf)
    vb = workload.bf16_normal(1403, (2, S, Hkv, d))
    kg, vg = (workload.bf16_normal(s, (Tq, Hkv, d)) for s in (1404, 1405))
    _run_and_check(qb, kg, vg, 0, kb, vb, "packed, far larger later score")


@pytest.mark.parametrize("Tq,G", [
    (40, 530),   # nine ranges of the generation shard, 64 rows each
    (33, 0),     # two ranges, the last of one row
    (8, 300),    # decode step: three ranges of up to 128 rows
    (4, 61),     # 64 rows a range at least: a second range of one row
])
def test_generation_ranges_follow_the_tokens(Tq, G):
    q = workload.bf16_normal(1500 + Tq, (Tq, 32, 128))
    kg, vg = (workload.bf16_normal(s + Tq, (G + Tq, 8, 128)) for s in (1501, 1502))
    k, v = (workload.bf16_normal(s + Tq, (2, 600, 8, 128)) for s in (1503, 1504))
    _run_and_check(q, kg, vg, G, k, v, f"generation ranges Tq={Tq} G={G}")


def test_workspace_sized_once_serves_smaller_steps():
    # a loop sizes its workspace for its largest step; every smaller one, on
    # whatever kernel and ranges, finds room in it
    H, S, Hq, Hkv, d, G = 3, 700, 32, 8, 128, 1200
    size = P.api._lib.lib().pulsar_phase2_query_workspace_bytes(H, 40, S, G, Hq, Hkv, d)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(5)
    def rows(*shape):
        return torch.randn(shape, generator=g, device="cuda").bfloat16()
    k, v = rows(H, S, Hkv, d), rows(H, S, Hkv, d)
    kg, vg = rows(G + 40, Hkv, d), rows(G + 40, Hkv, d)
    lib, ptr = P.api._lib.lib(), torch.Tensor.data_ptr
    for Tq in (1, 3, 8, 9, 20, 32, 33, 40):
        for g0 in (0, 31, 257, 1100, 1200):
            for h, s in ((1, 64), (1, 513), (2, 700), (3, 65), (3, 512), (3, 700)):
                q, kc, vc = rows(Tq, Hq, d), k[:h, :s].contiguous(), v[:h, :s].contiguous()
                o = torch.empty((Tq, Hq, d), device="cuda")
                lse = torch.empty((Hq, Tq), device="cuda")
                assert lib.pulsar_phase2_query(
                    ptr(q), ptr(kg), ptr(vg), g0, ptr(kc), ptr(vc), h, Tq, s, Hq, Hkv, d, 0.1,
                    ptr(o), ptr(lse), ptr(ws), size, P.api._stream()) == 0, (Tq, g0, h, s)
                ref = P.phase2_query(q, kg[:g0 + Tq], vg[:g0 + Tq], g0, kc, vc, softmax_scale=0.1)
                assert torch.equal(o, ref[0]) and torch.equal(lse, ref[1]), (Tq, g0, h, s)


@pytest.mark.parametrize("H,S,most,steps", [
    (1, 8192, 129, (128, 65, 64, 33, 1)),   # fewer row tiles take more key splits
    (3, 10846, 172, (109, 9, 8)),           # and more generation ranges
])
def test_workspace_of_the_attention_kernel_serves_smaller_steps(H, S, most, steps):
    Hq, Hkv, d = 32, 8, 128
    size = P.api._lib.lib().pulsar_phase2_query_workspace_bytes(H, most, S, 0, Hq, Hkv, d)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(6)
    def rows(*shape):
        return torch.randn(shape, generator=g, device="cuda").bfloat16()
    k, v = rows(H, S, Hkv, d), rows(H, S, Hkv, d)
    lib, ptr = P.api._lib.lib(), torch.Tensor.data_ptr
    for Tq in (most,) + steps:
        for h in range(1, H + 1):
            q, kg, vg = rows(Tq, Hq, d), rows(Tq, Hkv, d), rows(Tq, Hkv, d)
            o = torch.empty((Tq, Hq, d), device="cuda")
            lse = torch.empty((Hq, Tq), device="cuda")
            assert lib.pulsar_phase2_query(
                ptr(q), ptr(kg), ptr(vg), 0, ptr(k), ptr(v), h, Tq, S, Hq, Hkv, d, 0.1,
                ptr(o), ptr(lse), ptr(ws), size, P.api._stream()) == 0, (Tq, h)
            ref = P.phase2_query(q, kg, vg, 0, k[:h], v[:h], softmax_scale=0.1)
            assert torch.equal(o, ref[0]) and torch.equal(lse, ref[1]), (Tq, h)
    torch.cuda.synchronize()
