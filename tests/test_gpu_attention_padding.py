"""Waves whose 32 rows are all padding load and meet the others but compute
nothing: row counts on both sides of each wave's 32 rows, with and without
the key-split waves, one tile to many, tails of NaN, the overflow rerun (which
the idle waves must follow barrier by barrier), and block flags that leave
some waves of a tile without rows; against the oracle, both V layouts."""
import pytest
import torch

import oracle
import synth
import test_gpu_attention as A
from gpu_util import assert_attn_close, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# rows per KV head = group * window: 1 .. 128 run the key-split waves (32 rows
# for two waves), more the others; 33 and 288 put one row into a wave
@pytest.mark.parametrize("group,W,block", [(1, 1, 1), (1, 32, 32), (1, 33, 33), (4, 16, 16), (1, 96, 32), (4, 40, 8),
                                           (1, 160, 32), (4, 64, 32), (1, 257, 1), (4, 72, 8), (4, 96, 32)])
@pytest.mark.parametrize("D", [64, 128])
def test_row_counts(gpu, group, W, block, D):
    spec = synth.AttnSpec(3, block, 1, ("fixed", 0), 2 * group, 2, D)
    case = synth.make_attention_case(spec, 41, prefix_lens=[0, 77, 900], window_lens=[W, W, W], tail_fill=float("nan"),
                                     v_token_major=(group * W) % 3 == 0)
    say(f"  group {group} W {W} D {D}")
    for mode in ("bidir", "block_causal"):
        for split in (0, 128):
            out = A.run_case(gpu, case, mode, kv_split_tokens=split)
            assert_attn_close(out, A.oracle_case(case, mode), f"rows {group * W} D {D} {mode} split {split}")


@pytest.mark.parametrize("W", [8, 16, 40, 72, 96])
@pytest.mark.parametrize("mode", ["bidir", "block_causal"])
@pytest.mark.parametrize("vt", [False, True])
def test_overflow_rerun_beside_idle_waves(gpu, W, mode, vt):
    spec = synth.AttnSpec(3, 8, 1, ("fixed", 0), 16, 4, 128)
    case = synth.make_attention_case(spec, 53, prefix_lens=[700, 3000, 96], window_lens=[W] * 3, v_token_major=vt)
    case = A._plant_hot_keys(case, 54)
    for split in (0, 256):
        out = A.run_case(gpu, case, mode, kv_split_tokens=split)
        assert_attn_close(out, A.oracle_case(case, mode), f"rerun W={W} {mode} split={split}")


@pytest.mark.parametrize("mode", ["bidir", "block_causal"])
def test_block_flags_leave_waves_idle(gpu, mode):
    """Every pattern of flags over four blocks of 32 (256 rows of a tile are
    two blocks): tiles with no, one or both halves flagged."""
    B, k = 32, 4
    patterns = torch.tensor([[(i >> j) & 1 for j in range(k)] for i in range(16)], dtype=torch.uint8)
    spec = synth.AttnSpec(16, B, k, ("fixed", 0), 16, 4, 128)
    case = synth.make_attention_case(spec, 7, prefix_lens=[100 + 37 * i for i in range(16)])
    c = case.to(DEV)
    out = torch.full_like(c.q, -5.0)
    gpu.window_attention(c.q, c.k_pages, c.v_pages, c.page_table, c.prefix_lens, c.window_lens, B, out=out, mask_mode=mode,
                         host_prefix_lens=case.prefix_lens, host_window_lens=case.window_lens,
                         block_flags=patterns.to(DEV))
    torch.cuda.synchronize()
    rows = patterns.bool().repeat_interleave(B, dim=1).reshape(-1)
    ref = torch.as_tensor(A.oracle_case(case, mode))
    got = out.cpu()
    assert bool((got[~rows] == -5.0).all()), "rows of unflagged blocks were written"
    assert_attn_close(got[rows], ref[rows].numpy(), f"flags {mode}")
