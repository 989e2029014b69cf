"""The fp32 matrix-instruction kernel at its edges: tiles of odd sizes, key blocks of 16 cut short, rows beyond
one workgroup's 16, query heads beyond 16 per KV head at decode, launches of four and of eight waves."""
import numpy as np
import pytest
import torch

from oracle import dbsa_oracle as orc
from paper_2503_08640_amd import binding as B
from paper_2503_08640_amd import synth
from gpu_util import assert_close, pool_f64, to_dev, to_f64

pytestmark = pytest.mark.gpu

# Scores are sums of D products of N(0, 1) values scaled by 1/sqrt(D): absolute error at most about
# D * 2^-24 * sqrt(D) * max|q k| / sqrt(D) < 2e-4 for D = 128 and rounding errors of one sign, 1e-6 as they occur;
# a probability inherits it relatively, the output (a mean of values below 5) absolutely times 5.
MAX_TOL, MEAN_TOL = 2e-5, 2e-6


@pytest.mark.parametrize("hq,hkv,d,sink,pool,groups,window,bm,bn", [
    (2, 2, 64, 4, 260, 2, 0, 64, 64),     # fewer workgroups than compute units: eight waves
    (20, 1, 64, 1, 150, 3, 1, 40, 24),    # 20 query heads of one KV head, key tiles of 24
    (3, 3, 128, 17, 500, 2, 1, 1, 1),     # one row and one key per tile
    (16, 4, 128, 33, 1800, 3, 2, 200, 100),  # more workgroups than compute units: four waves
    (4, 2, 128, 0, 97, 1, 0, 1000, 1000),    # tiles larger than the pool
])
def test_fp32_attention_at_the_edges_of_its_blocks(hq, hkv, d, sink, pool, groups, window, bm, bn):
    pc = synth.make_pool_case("f32", 7000 + pool, dtype="f32", n_q_heads=hq, n_kv_heads=hkv, head_dim=d, sink_len=sink,
                              pool_tokens=pool, demo_len_range=(8, 31), n_groups=groups, prev_window=window)
    sels = [[groups - 1], [], list(range(groups))]
    qc = synth.make_query_case("f32q", 7001 + pool, pc, n_queries=3, q_len=[16, 1, 45], selections=sels, n_decode=2)
    p = pc.pool
    k, v = to_dev(pc.k), to_dev(pc.v)
    q64, k64, v64 = pool_f64(pc)
    lay = B.dbsa_layout_build(p.sink_len, p.demo_offsets, p.group_demo_offsets, window, block_m=bm, block_n=bn)
    lse = torch.empty((hq, p.n_tokens), dtype=torch.float32, device="cuda")
    o = B.dbsa_preencode_attn(lay, to_dev(pc.q), k, v, pc.scale, lse=lse)
    assert_close(to_f64(o), orc.preencode_attn(q64, k64, v64, p.sink_len, p.demo_offsets, p.group_demo_offsets, pc.scale,
                                               window), "fp32 pre-encode", MAX_TOL, MEAN_TOL)
    assert torch.isfinite(lse).all()
    layq = B.dbsa_layout_build(p.sink_len, p.demo_offsets, p.group_demo_offsets, cu_qlens=qc.cu_qlens, sel_ptr=qc.sel_ptr,
                               sel_idx=qc.sel_idx, block_m=bm, block_n=bn)
    oq = B.dbsa_query_attn(layq, to_dev(qc.q), to_dev(qc.k), to_dev(qc.v), k, v, pc.scale)
    assert_close(to_f64(oq), orc.query_attn(synth.as_f64(qc.q), synth.as_f64(qc.k), synth.as_f64(qc.v), k64, v64, p.sink_len,
                                            p.demo_offsets, p.group_demo_offsets, qc.cu_qlens, qc.sel_ptr, qc.sel_idx,
                                            pc.scale), "fp32 query prefill", MAX_TOL, MEAN_TOL)
    self_len = (np.diff(qc.cu_qlens) + 2).astype(np.int32)
    od = B.dbsa_decode_attn(layq, to_dev(qc.dec_q[1]), to_dev(qc.k_cache), to_dev(qc.v_cache), torch.from_numpy(self_len).cuda(),
                            k, v, pc.scale)
    assert_close(to_f64(od), orc.decode_attn(synth.as_f64(qc.dec_q[1]), synth.as_f64(qc.k_cache), synth.as_f64(qc.v_cache),
                                             self_len, k64, v64, p.sink_len, p.demo_offsets, p.group_demo_offsets, qc.sel_ptr,
                                             qc.sel_idx, pc.scale), "fp32 decode step", MAX_TOL, MEAN_TOL)


def test_a_value_beyond_a_short_block_does_not_reach_the_result():
    """Keys past a segment's end share their block's operands with the segment's last key: an infinite value there must
    reach the row that sees it and no row of another Q tile, those of its own group among them.  (The 16 rows of one
    workgroup share the value as an operand, and where causality hides it from a row it meets a weight of zero.)"""
    pc = synth.make_pool_case("f32inf", 7100, dtype="f32", n_q_heads=2, n_kv_heads=1, head_dim=64, sink_len=5, pool_tokens=60,
                              demo_len_range=(8, 12), n_groups=2)
    p = pc.pool
    v = to_dev(pc.v)
    v[p.n_tokens - 1] = float("inf")   # seen by the last row only
    lay = B.dbsa_layout_build(p.sink_len, p.demo_offsets, p.group_demo_offsets, block_m=16, block_n=64)
    o = B.dbsa_preencode_attn(lay, to_dev(pc.q), to_dev(pc.k), v, pc.scale)
    q64, k64, v64 = pool_f64(pc)
    tile, last_group = int(lay.export()[0][:, 0].max()), int(p.group_token_bounds()[-2])
    assert last_group < tile < p.n_tokens - 1 and (p.n_tokens - last_group) % 16   # rows of the group in front of the last tile
    want = orc.preencode_attn(q64, k64, v64, p.sink_len, p.demo_offsets, p.group_demo_offsets, pc.scale)
    assert_close(to_f64(o)[:tile], want[:tile], "rows of the other tiles", MAX_TOL, MEAN_TOL)
    assert torch.isinf(o[-1]).all()
