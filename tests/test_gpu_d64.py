"""head_dim 64 on the pipelined kernels: workgroups of one, two and four waves, persistent and one per Q tile, whole
lists, lists cut to measure and split, ragged tails, and scores that outgrow the running maximum."""
import numpy as np
import pytest
import torch

from oracle import dbsa_oracle as orc
from paper_2503_08640_amd import binding as B
from paper_2503_08640_amd import synth
from gpu_util import assert_close, to_dev, to_f64, two_waves
from test_gpu_parity import _oracle_query, _query_setup, small_pool_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,block_m,pool,groups,sink,window", [
    (4, 1, 64, 1100, 3, 5, 1),       # four waves of 64 rows, one workgroup per Q tile
    (4, 2, 64, 900, 2, 64, 0),       # two waves
    (4, 4, 64, 1100, 3, 130, 2),     # one wave
    (4, 4, 32, 500, 2, 0, 0),        # one wave whose second row block has no head
    (32, 8, 64, 6200, 23, 64, 0),    # the same persistently: Q tiles of many short groups in one stream
    (16, 16, 128, 9000, 20, 4, 0),
    (16, 16, 64, 9000, 20, 4, 0),
    (32, 8, 64, 4400, 1, 64, 0),     # the longest list decides: persistently, one wave to a SIMD
    (16, 16, 128, 9000, 2, 4, 0),
])
def test_pre_encode_at_head_dim_64(hq, hkv, block_m, pool, groups, sink, window):
    pc = small_pool_case("d64pre", 7200 + pool + block_m, hq=hq, hkv=hkv, d=64, sink=sink, pool_tokens=pool, groups=groups,
                         lens=(8, 120), sigma=0.5, w=window)
    p = pc.pool
    n = p.n_tokens
    lay = B.dbsa_layout_build(p.sink_len, p.demo_offsets, p.group_demo_offsets, window, block_m=block_m, block_n=64)
    lse = torch.zeros((hq, n), device="cuda")
    o = B.dbsa_preencode_attn(lay, to_dev(pc.q), to_dev(pc.k), to_dev(pc.v), pc.scale, lse=lse)
    rows = np.arange(n) if n < 2000 else np.unique(np.concatenate([np.arange(140), np.arange(n - 140, n),
                                                                   np.random.default_rng(1).integers(0, n, 400)]))
    want, want_lse = orc.preencode_attn(synth.as_f64(pc.q), synth.as_f64(pc.k), synth.as_f64(pc.v), p.sink_len, p.demo_offsets,
                                        p.group_demo_offsets, pc.scale, window, rows=rows, return_lse=True)
    assert_close(to_f64(o)[rows], want, f"d64 pre-encode {hq}/{hkv} bm={block_m}")
    assert_close(to_f64(lse)[:, rows], want_lse, "d64 lse")
    # every other row: V = 1 gives 1, up to the rounding of the probabilities (2^-9) and of the output (2^-9)
    one = B.dbsa_preencode_attn(lay, to_dev(pc.q), to_dev(pc.k), torch.ones_like(to_dev(pc.v)), pc.scale)
    assert (one.float() - 1).abs().max().item() <= 2.0 ** -8


@pytest.mark.parametrize("hq,hkv,block_m,q_len", [
    (8, 2, 64, [64]), (8, 2, 64, [1, 130, 64, 20, 77]), (8, 2, 32, [31, 5, 32]), (4, 4, 64, [150, 64, 9]), (4, 4, 256, [700, 90]),
])
def test_query_prefill_at_head_dim_64(hq, hkv, block_m, q_len):
    pc = small_pool_case("d64q", 7300 + block_m + len(q_len), hq=hq, hkv=hkv, d=64, pool_tokens=9000, groups=3, lens=(32, 200),
                         sigma=0.5)
    sels = [[2, 0], [0, 1, 2], [1], [], [2, 1, 0]][:len(q_len)]
    qc = synth.make_query_case("d64qq", 7301, pc, n_queries=len(q_len), q_len=q_len, selections=sels)
    lay, kp, vp = _query_setup(pc, qc, block_m, 0)
    qs, ks, vs = to_dev(qc.q), to_dev(qc.k), to_dev(qc.v)
    ref = _oracle_query(pc, qc)
    need = lay.workspace_bytes(hq, 64)
    outs = [B.dbsa_query_attn(lay, qs, ks, vs, kp, vp, pc.scale, workspace=ws)
            for ws in (False, torch.empty(need, dtype=torch.uint8, device="cuda"), torch.empty(need // 3, dtype=torch.uint8, device="cuda"))]
    for o, what in zip(outs, ("whole lists", "cut or split lists", "a third of the workspace")):
        assert_close(to_f64(o), ref, f"d64 {what} bm={block_m} T={q_len}")
    assert not torch.equal(outs[0], outs[1]), "the workspace changed nothing"


@pytest.mark.parametrize("hq,hkv,block_m,jump", [(8, 2, 64, 300.0), (4, 4, 64, 40.0), (4, 2, 64, 300.0)])
def test_scores_that_jump_at_head_dim_64(hq, hkv, block_m, jump):
    """Later keys of every segment score `jump` natural-log units above the first ones, for every row."""
    pc = small_pool_case("d64j", 7400 + hq, hq=hq, hkv=hkv, d=64, pool_tokens=2000, groups=3, lens=(32, 128))
    p = pc.pool
    k, q = to_dev(pc.k).float(), to_dev(pc.q).float()
    b = p.group_token_bounds()
    pos = np.concatenate([np.arange(p.sink_len)] + [np.arange(b[g + 1] - b[g]) for g in range(p.n_groups)])
    lift = torch.from_numpy((pos // 97).astype(np.float32)).cuda()
    q[..., 0] = 4.0
    k[..., 0] = lift[:, None] * (jump / (pc.scale * 4.0))
    q, k = q.bfloat16(), k.bfloat16()
    lay = B.dbsa_layout_build(p.sink_len, p.demo_offsets, p.group_demo_offsets, block_m=block_m, block_n=64)
    o = B.dbsa_preencode_attn(lay, q, k, to_dev(pc.v), pc.scale)
    assert_close(to_f64(o), orc.preencode_attn(to_f64(q), to_f64(k), synth.as_f64(pc.v), p.sink_len, p.demo_offsets,
                                               p.group_demo_offsets, pc.scale), f"d64 jump {jump}")


@pytest.mark.parametrize("hq,hkv,d,n_queries,n_split", [
    (8, 2, 64, 4, 0), (4, 4, 64, 40, 0), (16, 2, 64, 70, 0),     # one, two and four waves per workgroup
    (6, 2, 64, 5, 3), (6, 2, 128, 5, 0), (10, 2, 128, 45, 0), (7, 1, 128, 33, 0), (24, 1, 128, 3, 0),   # head ratios 3, 5, 7, 24
    (12, 1, 128, 40, 0),                                          # 12: a multiple of four that is no power of two
])
def test_group_major_decode_at_head_dim_64_and_odd_head_ratios(hq, hkv, d, n_queries, n_split):
    pc = small_pool_case("gmd", 7500 + hq + d, hq=hq, hkv=hkv, d=d, sink=70, pool_tokens=5000, groups=5, lens=(30, 200), sigma=0.5)
    sels = ([[3, 0], [], [4, 1, 2, 0, 3]] + [[1, 4]] * n_queries)[:n_queries]
    qc = synth.make_query_case("gmdq", 7501, pc, n_queries=n_queries, q_len=([64, 37, 100] + [9] * n_queries)[:n_queries],
                               selections=sels, n_decode=2)
    p = pc.pool
    lay = B.dbsa_layout_build(p.sink_len, p.demo_offsets, p.group_demo_offsets, cu_qlens=qc.cu_qlens, sel_ptr=qc.sel_ptr,
                              sel_idx=qc.sel_idx, n_split=n_split, block_m=32, block_n=64)
    shp = qc.k_cache.shape
    kc, vc = to_dev(qc.k_cache.reshape(-1, hkv, d)).view(shp), to_dev(qc.v_cache.reshape(-1, hkv, d)).view(shp)
    for s in range(2):   # (the second step walks the runs backwards)
        self_len = (np.diff(qc.cu_qlens) + s + 1).astype(np.int32)
        od = B.dbsa_decode_attn(lay, to_dev(qc.dec_q[s]), kc, vc, torch.from_numpy(self_len).cuda(), to_dev(pc.k), to_dev(pc.v),
                                pc.scale)
        ref = orc.decode_attn(synth.as_f64(qc.dec_q[s]), synth.as_f64(qc.k_cache), synth.as_f64(qc.v_cache), self_len,
                              synth.as_f64(pc.k), synth.as_f64(pc.v), p.sink_len, p.demo_offsets, p.group_demo_offsets,
                              qc.sel_ptr, qc.sel_idx, pc.scale)
        assert_close(to_f64(od), ref, f"decode {hq}/{hkv}x{d} {n_queries} queries step {s}")


@pytest.mark.parametrize("hq,hkv,d,block_m,pool", [
    (6, 2, 128, 64, 1500), (10, 2, 128, 64, 1500), (7, 1, 128, 32, 1500), (3, 1, 128, 128, 1500),   # one workgroup per Q tile
    (6, 2, 64, 64, 1500), (5, 1, 64, 32, 1500),
    (24, 8, 128, 64, 6200), (40, 8, 128, 64, 4000),                                                # persistent
])
def test_prefill_at_head_ratios_that_leave_waves_idle(hq, hkv, d, block_m, pool):
    pc = small_pool_case("odd", 7600 + hq + d + block_m, hq=hq, hkv=hkv, d=d, sink=70, pool_tokens=pool, groups=3 if pool < 2000 else 20,
                         lens=(20, 110), sigma=0.5)
    p = pc.pool
    n = p.n_tokens
    lay = B.dbsa_layout_build(p.sink_len, p.demo_offsets, p.group_demo_offsets, block_m=block_m, block_n=64)
    lse = torch.zeros((hq, n), device="cuda")
    guard = torch.full((n, hq + 1, d), 7.0, dtype=torch.bfloat16, device="cuda")   # one head more than the call may write
    o = B.dbsa_preencode_attn(lay, to_dev(pc.q), to_dev(pc.k), to_dev(pc.v), pc.scale, out=guard[:, :hq], lse=lse)
    rows = np.arange(n) if n < 2000 else np.unique(np.concatenate([np.arange(140), np.arange(n - 140, n),
                                                                   np.random.default_rng(2).integers(0, n, 300)]))
    want, want_lse = orc.preencode_attn(synth.as_f64(pc.q), synth.as_f64(pc.k), synth.as_f64(pc.v), p.sink_len, p.demo_offsets,
                                        p.group_demo_offsets, pc.scale, rows=rows, return_lse=True)
    assert_close(to_f64(o)[rows], want, f"pre-encode {hq}/{hkv}x{d} bm={block_m}")
    assert_close(to_f64(lse)[:, rows], want_lse, "lse")
    assert (guard[:, hq] == 7.0).all()
    qc = synth.make_query_case("oddq", 7601, pc, n_queries=3, q_len=[64, 100, 9], n_select=2)
    layq, kp, vp = _query_setup(pc, qc, block_m, 0)
    qs, ks, vs = to_dev(qc.q), to_dev(qc.k), to_dev(qc.v)
    for ws in (False, None):
        oq = B.dbsa_query_attn(layq, qs, ks, vs, kp, vp, pc.scale, workspace=ws)
        assert_close(to_f64(oq), _oracle_query(pc, qc), f"query prefill {hq}/{hkv}x{d} bm={block_m} ws={ws}")


def test_a_scale_whose_reciprocal_is_infinite_at_head_dim_64():
    """Any positive scale is taken: with one below 2^-128 all scores are zero to every digit, and a row is the mean of the
    values it sees."""
    pc = small_pool_case("d64t", 7700, hq=4, hkv=2, d=64, pool_tokens=700, groups=2, lens=(32, 128))
    p = pc.pool
    lay = B.dbsa_layout_build(p.sink_len, p.demo_offsets, p.group_demo_offsets, block_m=64, block_n=64)
    o = B.dbsa_preencode_attn(lay, to_dev(pc.q), to_dev(pc.k), to_dev(pc.v), 1e-39)
    want = orc.preencode_attn(synth.as_f64(pc.q), synth.as_f64(pc.k), synth.as_f64(pc.v), p.sink_len, p.demo_offsets,
                              p.group_demo_offsets, 1e-39)
    assert_close(to_f64(o), want, "d64 with a scale of 1e-39")


@pytest.mark.parametrize("hq,hkv,block_m,pool,groups,jump", [
    (32, 8, 64, 3600, 6, 0.0), (32, 8, 64, 3600, 6, 300.0), (32, 8, 64, 8800, 20, 0.0),     # four waves: one Q tile each, several
    (16, 16, 128, 7200, 12, 0.0), (16, 16, 128, 7200, 12, 40.0), (16, 16, 128, 16900, 20, 0.0),   # two waves
])
def test_encoding_with_two_waves_to_a_simd(hq, hkv, block_m, pool, groups, jump):
    """Launches that take two waves to a SIMD, dealt by a schedule and (first call under capture) in launch order; jump: as
    in the test of scores that jump."""
    pc = small_pool_case("d64crowd", 7800 + pool, hq=hq, hkv=hkv, d=64, sink=70, pool_tokens=pool, groups=groups, lens=(20, 120),
                         sigma=0.5)
    p = pc.pool
    n = p.n_tokens
    q, k, v = to_dev(pc.q).float(), to_dev(pc.k).float(), to_dev(pc.v)
    if jump:
        b = p.group_token_bounds()
        pos = np.concatenate([np.arange(p.sink_len)] + [np.arange(b[g + 1] - b[g]) for g in range(p.n_groups)])
        q[..., 0] = 4.0
        k[..., 0] = torch.from_numpy((pos // 97).astype(np.float32)).cuda()[:, None] * (jump / (pc.scale * 4.0))
    q, k = q.bfloat16(), k.bfloat16()
    lay = B.dbsa_layout_build(p.sink_len, p.demo_offsets, p.group_demo_offsets, block_m=block_m, block_n=64)
    assert two_waves(lay, 64) and (len(lay.export()[0]) <= 64) == (groups < 20)
    lse = torch.zeros((hq, n), device="cuda")
    o = B.dbsa_preencode_attn(lay, q, k, v, pc.scale, lse=lse)
    fresh = B.dbsa_layout_build(p.sink_len, p.demo_offsets, p.group_demo_offsets, block_m=block_m, block_n=64)
    unscheduled = torch.zeros_like(o)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.dbsa_preencode_attn(fresh, q, k, v, pc.scale, out=unscheduled)
    for _ in range(2):
        unscheduled.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(unscheduled, o), f"d64 crowded {hq}/{hkv} in launch order"
    rows = np.unique(np.concatenate([np.arange(140), np.arange(n - 140, n), np.random.default_rng(3).integers(0, n, 200)]))
    want, want_lse = orc.preencode_attn(to_f64(q), to_f64(k), to_f64(v), p.sink_len, p.demo_offsets, p.group_demo_offsets, pc.scale,
                                        rows=rows, return_lse=True)
    assert_close(to_f64(o)[rows], want, f"d64 crowded {hq}/{hkv} jump={jump}")
    if not jump:
        assert_close(to_f64(lse)[:, rows], want_lse, "d64 crowded lse")
    one = B.dbsa_preencode_attn(lay, q, k, torch.ones_like(v), pc.scale)
    assert (one.float() - 1).abs().max().item() <= 2.0 ** -8


@pytest.mark.parametrize("block_m,n_queries,top", [(64, 52, 64), (64, 30, 150), (32, 104, 20)])
def test_query_prefill_with_two_waves_to_a_simd(block_m, n_queries, top):
    """Questions for four fifths of two workgroups per SIMD and more, whole lists and (67 Q tiles) lists cut to measure."""
    pc = small_pool_case("d64crowdq", 7900 + block_m, hq=32, hkv=8, d=64, sink=70, pool_tokens=2600, groups=3, lens=(32, 120), sigma=0.5)
    rng = np.random.default_rng(5)
    q_len = [int(x) for x in rng.integers(max(1, top // 2), top + 1, size=n_queries)]
    sels = [[int(g) for g in rng.permutation(3)[:2]] for _ in range(n_queries)]
    qc = synth.make_query_case("d64crowdqq", 7901, pc, n_queries=n_queries, q_len=q_len, selections=sels)
    lay, kp, vp = _query_setup(pc, qc, block_m, 0)
    assert two_waves(lay, 4096 // block_m, False) and two_waves(lay, 4096 // block_m, True)
    qs, ks, vs = to_dev(qc.q), to_dev(qc.k), to_dev(qc.v)
    ref = _oracle_query(pc, qc)
    for ws in (False, None):
        assert_close(to_f64(B.dbsa_query_attn(lay, qs, ks, vs, kp, vp, pc.scale, workspace=ws)), ref, f"crowded queries ws={ws}")
