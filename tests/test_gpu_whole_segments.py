"""The decode kernel's choice of shares, at the sizes where it can go wrong.

Without a forced share count the kernel gives each workgroup one whole (sequence, KV
head) segment when there is a workgroup for each and none is much longer than an equal
share, and otherwise cuts the list into equal shares, fewer of them when segments would
fall into many pieces.  The lengths below put calls on each side: fewer pages than waves,
last pages of 1 and 16 tokens, more than 64 pages per wave (a second chunk of page ids),
as many segments as workgroups and one more, a long segment among short ones, one
segment alone.  Every output is compared with the fp64 oracle; the multi-token and the
packed grouped call take the same choice.
"""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2607_09207_amd import inputs as I
from test_gpu_grouped import run_grouped
from test_gpu_multi import run_multi
from test_gpu_parity import TOL, assert_close, gpu_run, torch_cuda  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu

CASES = {
    # pages per segment below, at and above the four waves; empty sequences between
    "few_pages_bf16": ("bf16", 28, 4, 128, [1, 16, 17, 0, 33, 48, 64, 65, 80, 0, 128]),
    "few_pages_fp8": ("fp8_e4m3fn", 40, 8, 128, [1, 16, 17, 0, 64, 65, 81]),
    "few_pages_d64": ("bf16", 16, 16, 64, [1, 15, 49, 256, 0, 257]),
    "few_pages_f32": ("f32", 4, 2, 64, [1, 16, 17, 0, 64, 65, 250]),
    # a segment for each workgroup (two a CU at d = 64: 512), and more segments than those
    "all_workgroups_bf16": ("bf16", 8, 8, 64, [40 + 7 * i for i in range(64)]),
    "more_segments_than_workgroups": ("bf16", 16, 16, 128, [20 + 3 * i for i in range(17)]),
    # more than 64 pages to a wave: equal long segments on three quarters of the workgroups
    "second_id_chunk_fp8": ("fp8_e4m3fn", 16, 16, 64, [4170 - i for i in range(24)]),
    # a long segment among short ones, and one or two segments alone (equal shares,
    # fewer than workgroups, many pieces)
    "one_long": ("bf16", 12, 2, 128, [9000, 5, 17, 300]),
    "alone_bf16": ("bf16", 8, 1, 128, [3001]),
    "alone_fp8": ("fp8_e4m3fn", 4, 2, 64, [12345]),
    "alone_f32": ("f32", 1, 1, 128, [2049]),
}


@pytest.mark.parametrize("out", ["f32", "bf16"])
@pytest.mark.parametrize("name", list(CASES))
def test_default_shares_match_the_oracle(torch_cuda, name, out):
    kv, Hq, Hkv, d, lens = CASES[name]
    if kv == "f32" and out == "bf16":
        pytest.skip("fp32 caches have fp32 outputs")
    w = I.make_custom(lens, Hq, Hkv, d, q_dtype="f32" if kv == "f32" else "bf16", kv_dtype=kv, seed=71, extra_pages=2)
    got, flags = gpu_run(torch_cuda, w, out_dtype=out, tag=f"shares {name}")
    assert flags == 0
    assert_close(got, oracle.run(w), kv, f"shares {name} out={out}")


@pytest.mark.parametrize("kv,d,G", [("bf16", 128, 7), ("bf16", 64, 4), ("fp8_e4m3fn", 128, 5)])
def test_default_shares_of_multi_token_rows(torch_cuda, kv, d, G):
    lens = [5, 16, 17, 200, 64, 333, 1]
    w = I.make_multi(lens, [min(L, 4) for L in lens], 2 * G, 2, d, kv_dtype=kv, seed=72, extra_pages=1)
    got, flags = run_multi(torch_cuda, w, max_q_len=4)
    assert flags == 0
    assert np.max(np.abs(got - oracle.run_multi(w))) <= TOL[kv]


@pytest.mark.parametrize("prompt", [32, 512])
def test_default_shares_of_packed_groups(torch_cuda, prompt):
    tails = [1, 16, 17, 40, 0, 300, 33, 5]
    w = I.make_custom([prompt + t for t in tails], 12, 2, 128, seed=73, shared_prefix=(4, prompt), extra_pages=1)
    got, flags = run_grouped(torch_cuda, w, 4, [prompt // 16] * 2)
    assert flags == 0
    assert_close(got, oracle.run(w), "bf16", f"packed prompt={prompt}")


@pytest.mark.parametrize("name", ["few_pages_bf16", "few_pages_fp8", "few_pages_d64", "second_id_chunk_fp8"])
def test_whole_segments_keep_the_probabilities_remainders(torch_cuda, name):
    """A probability and its bf16 remainder carry 16 bits (relative error 2^-17 each), so an
    output is off by at most 2^-17 max|v|; fp32 scores and sums of up to 4170 keys add less
    than that again.  Without the remainders the error is about 2^-9 max|v| / sqrt(keys)."""
    kv, Hq, Hkv, d, lens = CASES[name]
    w = I.make_custom(lens, Hq, Hkv, d, kv_dtype=kv, seed=74, extra_pages=2)
    got, flags = gpu_run(torch_cuda, w, tag=f"remainders {name}")
    assert flags == 0
    worst = float(np.max(np.abs(got - oracle.run(w))))
    assert worst <= 2.0 ** -16 * 6.0, worst   # |v| < 6: normal values


# As many segments as workgroups on 256 CUs, and one more: (dtype, d, KV heads, sequences).
EDGE = {"full_256": ("bf16", 128, 1, 256), "full_257": ("bf16", 128, 1, 257),
        "half_512": ("bf16", 64, 2, 256), "half_513": ("bf16", 64, 3, 171),
        "fp8_512": ("fp8_e4m3fn", 128, 2, 256), "fp8_513": ("fp8_e4m3fn", 128, 3, 171)}


@pytest.mark.parametrize("name", list(EDGE))
def test_as_many_segments_as_workgroups_and_one_more(torch_cuda, name):
    """Whole segments up to there, W equal shares (no remainders) above: the error tells."""
    from paper_2607_09207_amd import calibrate
    cus = torch_cuda.cuda.get_device_properties(0).multi_processor_count
    if cus != 256:
        pytest.skip("the sequence counts are for 256 CUs")
    kv, d, hkv, n = EDGE[name]
    w = I.make_custom([40 + i % 60 for i in range(n)], 4 * hkv, hkv, d, kv_dtype=kv, seed=77, extra_pages=2)
    workgroups = cus if name.startswith("full") else 2 * cus
    whole, shares = calibrate.work_split(w.seq_lens, hkv, workgroups, d, kv)
    assert (whole, shares) == ((True, shares) if n * hkv <= workgroups else (False, workgroups))
    got, flags = gpu_run(torch_cuda, w, tag=f"edge {name}")
    assert flags == 0
    want = oracle.run(w)
    assert_close(got, want, kv, f"edge {name}")
    worst = float(np.max(np.abs(got - want)))
    assert (worst <= 2.0 ** -16 * 6.0) == whole, worst


# The other calls that get longer streams than one equal share a workgroup: rows of several
# query tokens, packed groups, the attention launch after a (zero) prompt pass, and few
# segments in fewer shares.
LONGER = {
    # (Hq, Hkv, lengths, query rows, group size, prompt tokens)
    "rows_one_tile": (8, 2, [640, 200, 333, 17], 4, 0, 0),
    "rows_two_tiles": (8, 1, [640, 200, 333, 17], 4, 0, 0),
    "packed": (12, 2, [144, 200, 133, 129, 300, 128, 177, 190], 0, 4, 128),
    "after_prompt_pass": (16, 1, [300, 17, 555, 100], 0, 4, 0),
    "fewer_shares_one_segment": (8, 1, [3001], 0, 0, 0),
    "fewer_shares_ragged": (12, 2, [9000, 5, 17, 300], 0, 0, 0),
}


def longer_call(torch, name, kv, d, change=None):
    """The call's output, its flags and the oracle's output; `change` alters the inputs."""
    Hq, Hkv, lens, rows, group, prompt = LONGER[name]
    if rows:
        w = I.make_multi(lens, [min(L, rows) for L in lens], Hq, Hkv, d, kv_dtype=kv, seed=76)
    else:
        w = I.make_custom(lens, Hq, Hkv, d, kv_dtype=kv, seed=76, shared_prefix=(group, prompt) if prompt else None)
    w = change(w) if change else w
    if rows:
        return run_multi(torch, w, max_q_len=rows) + (oracle.run_multi(w),)
    if group:
        return run_grouped(torch, w, group, [prompt // 16] * (w.batch // group)) + (oracle.run(w),)
    return gpu_run(torch, w, tag=name) + (oracle.run(w),)


@pytest.mark.parametrize("kv,d", [("bf16", 128), ("bf16", 64), ("fp8_e4m3fn", 128), ("fp8_e4m3fn", 64)])
@pytest.mark.parametrize("name", list(LONGER))
def test_longer_streams_keep_the_remainders_too(torch_cuda, name, kv, d):
    got, flags, want = longer_call(torch_cuda, name, kv, d)
    assert flags == 0
    worst = float(np.max(np.abs(got - want)))
    assert worst <= 2.0 ** -16 * 6.0, worst   # as above


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("name", list(LONGER))
def test_infinite_values_in_longer_streams(torch_cuda, name, d):
    """Infinities among the first keys, which every row of the call sees."""
    def change(w):
        v = w.v_cache.copy()
        for b in np.flatnonzero(w.seq_lens > 16):
            for token, col, bits in ((0, 5, 0x7F80), (9, 6, 0xFF80), (3, 9, 0x7F80), (8, 9, 0xFF80)):
                v[w.block_table[b, 0], :, token, col] = bits
        return dataclasses.replace(w, v_cache=v)

    got, flags, want = longer_call(torch_cuda, name, "bf16", d, change)
    assert flags == 0
    finite = np.isfinite(want)
    assert np.isposinf(want).any() and np.isneginf(want).any() and np.isnan(want).any()
    assert np.array_equal(got[~finite], want[~finite], equal_nan=True)
    assert np.max(np.abs(got[finite] - want[finite])) <= TOL["bf16"]


@pytest.mark.parametrize("name", ["few_pages_bf16", "few_pages_d64"])
def test_infinite_values_stay_infinite(torch_cuda, name):
    """An infinite V times a probability is that infinity, whatever share of a call its
    sequence gets (0 times it, or two of unlike sign, would be NaN): the outputs are
    infinite, NaN and finite where the oracle's are."""
    kv, Hq, Hkv, d, lens = CASES[name]
    w = I.make_custom(lens, Hq, Hkv, d, kv_dtype=kv, seed=75, extra_pages=2)
    v, PINF, NINF = w.v_cache.copy(), 0x7F80, 0xFF80
    for b in np.flatnonzero(w.seq_lens > 16):
        for token, col, bits in ((0, 5, PINF), (9, 6, NINF), (w.seq_lens[b] - 1, 7, PINF), (3, 9, PINF), (16, 9, NINF)):
            v[w.block_table[b, token // 16], :, token % 16, col] = bits
    w = dataclasses.replace(w, v_cache=v)
    want = oracle.run(w)
    finite = np.isfinite(want)
    assert np.isposinf(want).any() and np.isneginf(want).any() and np.isnan(want).any()
    for ranges in (0, 5):
        got, flags = gpu_run(torch_cuda, w, ranges=ranges, tag=f"infinite {name}")
        assert flags == 0
        assert np.array_equal(got[~finite], want[~finite], equal_nan=True), f"ranges={ranges}"
        assert np.max(np.abs(got[finite] - want[finite])) <= TOL[kv]
