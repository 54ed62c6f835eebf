"""The attention kernel for units of at most four key tiles: key counts on both
sides of its tiles and in its 1- to 4-tile forms, row counts on both sides of
a wave's and a workgroup's rows, one split and many, ragged lengths (dispatch
table), bounds only, NaN tails, block flags and the gate; against the oracle,
and against the general kernel over random shapes of the range."""
import numpy as np
import pytest
import torch

import synth
import test_gpu_attention as A
from gpu_util import assert_attn_close, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _plan(gpu, c, **kw):
    return gpu.window_attention_plan(c.num_q_heads, c.k_pages, c.v_pages, c.page_table, c.batch, int(c.q.shape[0]),
                                     max_prefix_len=int(c.prefix_lens.max()), max_window_len=int(c.window_lens.max()),
                                     host_prefix_lens=c.prefix_lens, host_window_lens=c.window_lens, **kw)


@pytest.mark.parametrize("keys", [1, 15, 32, 33, 63, 64, 65, 127, 128, 129, 191, 193, 255, 256, 257, 400, 2100])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("vt", [False, True])
def test_key_counts(gpu, keys, D, vt):
    W = min(keys, 32)
    spec = synth.AttnSpec(2, W, 1, ("fixed", 0), 8, 2, D)
    case = synth.make_attention_case(spec, keys, prefix_lens=[keys - W, max(0, keys - W - 1)], window_lens=[W, W],
                                     tail_fill=float("nan"), v_token_major=vt)
    assert "short" in _plan(gpu, case)["kernel"]
    for mode in ("bidir", "block_causal"):
        assert_attn_close(A.run_case(gpu, case, mode), A.oracle_case(case, mode), f"keys {keys} D {D} vt {vt} {mode}")


@pytest.mark.parametrize("group,W,block", [(1, 1, 1), (1, 33, 33), (3, 11, 11), (4, 32, 16), (3, 43, 43), (4, 64, 32),
                                           (8, 48, 16), (4, 128, 32)])
@pytest.mark.parametrize("vt", [False, True])
def test_row_counts(gpu, group, W, block, vt):
    """1 to 512 rows per KV head: part of a wave, of a workgroup, several."""
    spec = synth.AttnSpec(2, block, 1, ("fixed", 0), 2 * group, 2, 128)
    case = synth.make_attention_case(spec, 3, prefix_lens=[77, 600], window_lens=[W, W], tail_fill=float("nan"),
                                     v_token_major=vt)
    assert "short" in _plan(gpu, case)["kernel"]
    for mode in ("bidir", "block_causal"):
        assert_attn_close(A.run_case(gpu, case, mode), A.oracle_case(case, mode), f"rows {group * W} vt {vt} {mode}")


@pytest.mark.parametrize("split", [64, 128, 192, 256])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("vt", [False, True])
def test_unit_lengths(gpu, split, D, vt):
    """One form per tile count of a unit, with a last unit of one key, of one tile
    less, and whole."""
    spec = synth.AttnSpec(4, 16, 1, ("fixed", 0), 8, 2, D)
    case = synth.make_attention_case(spec, split, prefix_lens=[2 * split + 1 - 16, 3 * split - 64, 3 * split - 16, 5],
                                     window_lens=[16] * 4, tail_fill=float("nan"), v_token_major=vt)
    kernel = _plan(gpu, case, kv_split_tokens=split)["kernel"]
    assert "short" in kernel and kernel.endswith(f",{split // 64}>"), kernel
    for mode in ("bidir", "block_causal"):
        assert_attn_close(A.run_case(gpu, case, mode, kv_split_tokens=split), A.oracle_case(case, mode),
                          f"units of {split} D {D} vt {vt} {mode}")


@pytest.mark.parametrize("seed", range(16))
def test_random_against_general_kernel(gpu, seed, monkeypatch):
    rng = np.random.default_rng(900 + seed)
    batch, hkv, group = int(rng.integers(1, 5)), int(rng.choice([1, 2, 4])), int(rng.choice([1, 2, 4]))
    D, B = int(rng.choice([64, 128])), int(rng.choice([8, 16, 32]))
    P = [int(x) for x in rng.integers(0, 1500 // batch, size=batch)]
    W = [int(x) * B for x in rng.integers(0, 4, size=batch)]
    W[0] = 2 * B
    spec = synth.AttnSpec(batch, B, 4, ("fixed", 0), hkv * group, hkv, D)
    case = synth.make_attention_case(spec, seed, prefix_lens=P, window_lens=W, tail_fill=float("nan"),
                                     v_token_major=bool(seed & 1))
    mode = ("bidir", "block_causal")[seed // 2 % 2]
    say(f"  seed {seed} batch {batch} heads {hkv}x{group} D {D} P {P} W {W} {mode}")
    assert "short" in _plan(gpu, case)["kernel"]
    out = A.run_case(gpu, case, mode).float().cpu()
    ref = A.oracle_case(case, mode)
    assert_attn_close(out, ref, f"short {seed}")
    monkeypatch.setenv("MBE_ATTN_PIPELINE", "0")
    general = A.run_case(gpu, case, mode).float().cpu()
    assert_attn_close(out, general.double().numpy(), f"short against general {seed}")


@pytest.mark.parametrize("vt", [False, True])
def test_sharp_scores_and_late_maximum(gpu, vt):
    """Scores of hundreds of log2 units whose maximum comes late: the general
    kernel's rerun, here the ordinary path."""
    spec = synth.AttnSpec(3, 32, 2, ("fixed", 0), 16, 4, 128)
    case = synth.make_attention_case(spec, 53, prefix_lens=[700, 190, 96], v_token_major=vt)
    case = A._plant_hot_keys(case, 54)
    assert "short" in _plan(gpu, case)["kernel"]
    for mode in ("bidir", "block_causal"):
        assert_attn_close(A.run_case(gpu, case, mode), A.oracle_case(case, mode), f"sharp {mode}")


@pytest.mark.parametrize("mode", ["bidir", "block_causal"])
def test_flags_and_gate(gpu, mode):
    B, k = 32, 4
    patterns = torch.tensor([[(i >> j) & 1 for j in range(k)] for i in (0, 1, 6, 9, 15)], dtype=torch.uint8)
    spec = synth.AttnSpec(5, B, k, ("fixed", 0), 8, 2, 128)
    case = synth.make_attention_case(spec, 7, prefix_lens=[100 + 37 * i for i in range(5)])
    c = case.to(DEV)
    rows = patterns.bool().repeat_interleave(B, dim=1).reshape(-1)
    ref = torch.as_tensor(A.oracle_case(case, mode))
    for gate in (None, 0, 1):
        out = torch.full_like(c.q, -5.0)
        kw = {} if gate is None else {"run_if_nonzero": torch.tensor([gate], dtype=torch.int32, device=DEV)}
        gpu.window_attention(c.q, c.k_pages, c.v_pages, c.page_table, c.prefix_lens, c.window_lens, B, out=out,
                             mask_mode=mode, host_prefix_lens=case.prefix_lens, host_window_lens=case.window_lens,
                             block_flags=patterns.to(DEV), **kw)
        got = out.cpu()
        if gate == 0:
            assert bool((got == -5.0).all()), "a gated-off call wrote"
            continue
        assert bool((got[~rows] == -5.0).all()), "rows of unflagged blocks were written"
        assert_attn_close(got[rows], ref[rows].numpy(), f"flags {mode} gate {gate}")
