"""The split merge with 1, 2, 4 and 8 lanes per item (split counts on both
sides of each, ragged so that some sequences have fewer), and the refresh flags
around their 64 lanes, in place too."""
import numpy as np
import pytest
import torch

import synth
import test_gpu_attention as A
from gpu_util import assert_attn_close

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("nsplit", [2, 8, 9, 15, 16, 17, 25, 32, 33, 47, 64, 65, 130])
@pytest.mark.parametrize("D", [64, 128])
def test_merge_lanes(gpu, nsplit, D):
    n = nsplit * 64
    spec = synth.AttnSpec(3, 16, 2, ("fixed", 0), 6, 2, D)
    case = synth.make_attention_case(spec, nsplit, prefix_lens=[n - 32, n // 2, 1], window_lens=[32, 16, 32],
                                     tail_fill=float("nan"), v_token_major=nsplit % 2 == 1)
    for mode in ("bidir", "block_causal"):
        out = A.run_case(gpu, case, mode, kv_split_tokens=64)
        assert_attn_close(out, A.oracle_case(case, mode), f"{nsplit} splits D {D} {mode}")


@pytest.mark.parametrize("W,hq,nsplit", [(128, 32, 17), (64, 16, 33), (64, 16, 70), (32, 8, 70)])
def test_merge_lanes_of_many_splits(gpu, W, hq, nsplit):
    """More items than leave room for the lanes that would hold the splits: one, two
    (33 and 70 splits) and four lanes with more than 8 splits each."""
    n = nsplit * 64
    spec = synth.AttnSpec(3, 16, W // 16, ("fixed", 0), hq, 4, 128)
    case = synth.make_attention_case(spec, nsplit, prefix_lens=[n - W, n // 2, 1], window_lens=[W, 16, W],
                                     tail_fill=float("nan"))
    out = A.run_case(gpu, case, "bidir", kv_split_tokens=64)
    assert_attn_close(out, A.oracle_case(case, "bidir"), f"{nsplit} splits W {W} heads {hq}")


@pytest.mark.parametrize("num_blocks", [1, 4, 63, 64, 65, 130])
@pytest.mark.parametrize("mode", ["changed", "changed_and_later"])
def test_refresh_flags(gpu, num_blocks, mode):
    rng = np.random.default_rng(num_blocks)
    c = (rng.random((9, num_blocks)) < 2.0 / num_blocks).astype(np.uint8) * 3       # any nonzero value counts
    c[0] = 0
    c[1] = 0
    c[1, -1] = 1
    want = (c != 0).astype(np.uint8)
    if mode == "changed_and_later":
        want = np.maximum.accumulate(want, axis=1)
    d = torch.from_numpy(c).to(DEV)
    assert np.array_equal(gpu.refresh_blocks(d, mode).cpu().numpy(), want)
    gpu.refresh_blocks(d, mode, out=d)
    assert np.array_equal(d.cpu().numpy(), want)
