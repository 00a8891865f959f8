"""The attention kernel's fragment streams at the sizes where they turn: ranks
around whole rounds of slots (a run's odd steps, runs shorter than a round, every
split of the value pass), one to five 256-token tiles per block, column tiles of at
most 32 columns (one output slice per wave) and of more (two), workgroups that fold
several items into one group, gangs that fetch the coming tile into L2 and gangs
that do not, and items whose first run is of another kind than the last one's.
Against the fp64 oracle at the 1e-2 bar that bf16 operands with fp32 sums give
(three roundings of 2^-9 each, observed 3e-3 to 8e-3)."""
import numpy as np
import pytest

import oracle
import synth
from helpers import TOL_REL_L2, GpuLayer, max_rel_l2, oracle_args, oracle_args_int8

pytestmark = pytest.mark.gpu

CASES = {
    # ranks 32 .. 160: 2 .. 10 rank steps; 1 .. 5 tiles; a gang of one
    "short_runs": dict(block_tokens=[256, 300, 700, 1000, 1280], rank_k=[32, 64, 96, 128, 160],
                       rank_v=[160, 128, 96, 64, 32], n_kv_heads=2, head_dim=128, n_q=1, n_q_heads=8),
    # 64 columns (two heads of 32) and 33 columns per tile
    "cols_32": dict(block_tokens=[520, 256], rank_k=[200, 64], n_kv_heads=2, head_dim=128, n_q=4, n_q_heads=16),
    "cols_33": dict(block_tokens=[520, 256], rank_k=[50, 64], n_kv_heads=1, head_dim=64, n_q=3, n_q_heads=11),
    "cols_33_d128": dict(block_tokens=[520, 256], rank_k=[128, 120], n_kv_heads=1, head_dim=128, n_q=3, n_q_heads=11),
    # every split of the value pass, K and V ranks of different kinds in turn
    "splits": dict(block_tokens=[512] * 8, rank_k=[512, 32, 288, 250, 500, 17, 96, 384],
                   rank_v=[32, 64, 96, 160, 224, 256, 288, 512], n_kv_heads=4, head_dim=128, n_q=10, n_q_heads=28),
    # 768 and 784 columns over ragged blocks
    "cols_768": dict(block_tokens=[1100, 256, 513, 769], rank_k=[320, 96, 500, 40], n_kv_heads=8, head_dim=128,
                     n_q=24, n_q_heads=32),
    "cols_784": dict(block_tokens=[1100, 256, 513, 769], rank_k=[320, 96, 500, 40], n_kv_heads=8, head_dim=128,
                     n_q=14, n_q_heads=56),
    # above 512: three and four rank tiles per wave
    "ranks_544_896": dict(block_tokens=[1000, 900, 300], rank_k=[544, 896, 33], rank_v=[768, 520, 200], n_kv_heads=8,
                          head_dim=128, n_q=9, n_q_heads=16),
}


@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("p_int8", [False, True])
def test_streams(name, p_int8):
    kw = CASES[name]
    inp = synth.make_problem(7000 + sorted(CASES).index(name), tail_cap=9, **kw)
    gl = GpuLayer(inp, p_int8=p_int8)
    try:
        got = gl.attend().cpu().numpy()
        again = gl.attend().cpu().numpy()
    finally:
        gl.free()
    ref = oracle.attend_latent(**(oracle_args_int8(inp) if p_int8 else oracle_args(inp)))
    assert np.all(np.isfinite(got)) and np.array_equal(got, again)
    assert max_rel_l2(got, ref) <= TOL_REL_L2


MORE = {
    # tiles of 32 columns (four heads of 8), R^V of 4, 5, 8, 9 and 16 steps: one and two
    # rounds of the narrow up-projection and their remainders
    "narrow_32": dict(block_tokens=[520, 300, 1024, 700, 512], rank_k=[96, 160, 256, 288, 512],
                      rank_v=[128, 160, 256, 288, 512], n_kv_heads=4, head_dim=128, n_q=1, n_q_heads=32),
    "narrow_32_d64": dict(block_tokens=[520, 300, 1024, 700, 512], rank_k=[96, 160, 256, 288, 512],
                          rank_v=[128, 160, 256, 288, 512], n_kv_heads=8, head_dim=64, n_q=1, n_q_heads=64),
    # 36 columns (four heads of 9): two slices per wave over the same ranks
    "wide_36": dict(block_tokens=[520, 300, 1024, 700, 512], rank_k=[96, 160, 256, 288, 512],
                    rank_v=[128, 160, 256, 288, 512], n_kv_heads=4, head_dim=128, n_q=3, n_q_heads=12),
    # 600 one- and two-tile blocks of one column tile: each workgroup folds two or three
    # items into one partial, between tails, with waves that own no rank tile
    "fold": dict(block_tokens=[100, 256, 300] * 200, rank_k=[17, 64, 96] * 200, rank_v=[32, 96, 20] * 200,
                 n_kv_heads=2, head_dim=128, n_q=2, n_q_heads=10),
    "fold_d64": dict(block_tokens=[100, 256, 300] * 200, rank_k=[17, 64, 96] * 200, rank_v=[32, 96, 20] * 200,
                     n_kv_heads=2, head_dim=64, n_q=2, n_q_heads=10),
    # gangs of ten on either side of the mean rank (rk + rv = 320) from which they fetch
    "gang_low": dict(block_tokens=[1100, 256, 769, 1000], rank_k=[96, 250, 128, 100], n_kv_heads=8, head_dim=128,
                     n_q=16, n_q_heads=40),
    "gang_fetch": dict(block_tokens=[1100, 288, 769, 1000], rank_k=[320, 256, 500, 288], n_kv_heads=8, head_dim=128,
                       n_q=16, n_q_heads=40),
    # three and more tiles per part at d = 64, fetching, and rank tiles up to 512
    "gang_fetch_d64": dict(block_tokens=[1100, 900, 2000, 513], rank_k=[320, 288, 512, 480], n_kv_heads=8, head_dim=64,
                           n_q=16, n_q_heads=40),
    # one short block per workgroup and a gang of one at d = 64
    "single_d64": dict(block_tokens=[256, 200, 130], rank_k=[32, 100, 128], n_kv_heads=2, head_dim=64, n_q=1, n_q_heads=14),
}


@pytest.mark.parametrize("name", sorted(MORE))
@pytest.mark.parametrize("p_int8", [False, True])
def test_more_streams(name, p_int8):
    inp = synth.make_problem(7100 + sorted(MORE).index(name), tail_cap=9, **MORE[name])
    gl = GpuLayer(inp, p_int8=p_int8)
    try:
        got = gl.attend().cpu().numpy()
        again = gl.attend().cpu().numpy()
    finally:
        gl.free()
    ref = oracle.attend_latent(**(oracle_args_int8(inp) if p_int8 else oracle_args(inp)))
    assert np.all(np.isfinite(got)) and np.array_equal(got, again)
    assert max_rel_l2(got, ref) <= TOL_REL_L2
