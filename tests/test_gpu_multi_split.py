"""The forms of the MFMA multi-token call, at the sizes where they can go wrong.

A call of few row blocks takes either 128 rows to a workgroup or 32 with the keys dealt
to its four waves in blocks of 32; the kernel chooses from the lengths.  Other calls run
the 128-row kernel.  The lengths below leave waves without a block, end inside a page, a
block and a round of four blocks, take more than 32 blocks to a wave (page ids are fetched
32 blocks at a time) and hold more than 64 sequences (tables in LDS).  Every output is
compared with the fp64 oracle.
"""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2607_09207_amd import inputs as I
from test_gpu_multi import run_multi
from test_gpu_parity import assert_close, torch_cuda  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu

EDGES = [1, 2, 16, 17, 31, 32, 33, 255, 256, 257, 0, 1000]
CASES = {
    # few row blocks, at most two 32-row items a CU, 96 keys or more: the keys are split
    "edges_one_head": (8, 1, EDGES, [1, 1, 16, 5, 31, 32, 3, 100, 4, 257, 0, 33]),
    "edges_four_heads": (28, 4, EDGES, [1, 2, 1, 17, 3, 32, 33, 9, 40, 2, 0, 12]),
    "many_blocks_a_wave": (4, 2, [9001, 8192, 40], [5, 33, 40]),
    "above_64_sequences": (8, 1, [(37 * i) % 300 + 1 for i in range(90)], [1 + i % 2 for i in range(90)]),
    "eight_heads": (8, 8, [700, 65, 129], [130, 65, 1]),
    # more items than that: split from 640 keys on
    "two_rounds_split": (32, 8, [800, 700], [300, 300]),
    "two_rounds_whole": (32, 8, [230, 229, 230], [230, 229, 230]),
    # below 96 keys: 128 rows
    "short": (28, 4, [1, 2, 16, 17, 31, 32, 33, 95], [1, 2, 1, 17, 31, 3, 33, 95]),
    # many row blocks: the 128-row kernel
    "rows128_edges": (32, 16, EDGES + [600, 400, 300], [1, 2, 1, 17, 31, 32, 33, 255, 40, 257, 0, 300, 600, 400, 300]),
    "rows128_four_heads": (28, 4, EDGES + [600, 500], [1, 2, 1, 17, 31, 32, 33, 255, 40, 257, 0, 300, 600, 100]),
}


@pytest.mark.parametrize("kv,d", [("bf16", 128), ("bf16", 64), ("fp8_e4m3fn", 128), ("fp8_e4m3fn", 64)])
@pytest.mark.parametrize("name", list(CASES))
def test_both_forms_match_the_oracle(torch_cuda, name, kv, d):
    Hq, Hkv, lens, ql = CASES[name]
    w = I.make_multi(lens, ql, Hq, Hkv, d, q_dtype="bf16", kv_dtype=kv, seed=91, extra_pages=2)
    out = "bf16" if name == "eight_heads" else "f32"
    got, flags = run_multi(torch_cuda, w, out_dtype=out, tag=f"forms {name}")
    assert flags == 0
    assert_close(got, oracle.run_multi(w), kv, f"forms {name} {kv} d={d}")


@pytest.mark.parametrize("Hq,Hkv", [(8, 1), (64, 16)], ids=["split", "rows128"])
def test_fp8_pages_of_scale_zero(torch_cuda, Hq, Hkv):
    """A K or V page of scale 0 (all its values are 0) among others: scores of 0."""
    w = I.make_multi([400, 333, 90], [200, 333, 90], Hq, Hkv, 128, q_dtype="bf16", kv_dtype="fp8_e4m3fn", seed=92)
    ks, vs = np.array(w.k_scale), np.array(w.v_scale)
    ks[::3] = 0
    vs[::5] = 0
    w = dataclasses.replace(w, k_scale=ks, v_scale=vs)
    got, flags = run_multi(torch_cuda, w, tag=f"zero scales Hkv={Hkv}")
    assert flags == 0
    assert_close(got, oracle.run_multi(w), "fp8_e4m3fn", f"zero scales Hkv={Hkv}")


@pytest.mark.parametrize("Hq,Hkv", [(8, 1), (64, 16)], ids=["split", "rows128"])
def test_a_page_id_out_of_the_pool_spares_the_other_sequences(torch_cuda, Hq, Hkv):
    w = I.make_multi([400, 333, 90], [200, 333, 90], Hq, Hkv, 128, q_dtype="bf16", kv_dtype="bf16", seed=93)
    bt = np.array(w.block_table)
    bt[1, 7] = w.num_pages + 1000
    got, flags = run_multi(torch_cuda, dataclasses.replace(w, block_table=bt), tag=f"bad page Hkv={Hkv}")
    assert flags == 1
    want = oracle.run_multi(w)
    ok = np.r_[0:200, 533:623]
    assert_close(got[ok], want[ok], "bf16", f"bad page Hkv={Hkv}")
    assert np.all(np.isfinite(got))
