"""The per-block steps of one wave per block (at most 64 rows) and of one
workgroup per block (more) on both sides of that line, for block counts that
leave waves of the last workgroup without a block: the update against the
oracle with every kind of row (masked, confident, forced, tied, gated off), the
tail scores against a sort."""
import math

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("block", [1, 2, 3, 31, 32, 33, 63, 64, 65, 100])
@pytest.mark.parametrize("blocks", [1, 3, 4, 5, 30])
def test_update_blocks(gpu, block, blocks):
    rows, vocab = block * blocks, 600                     # (one chunk per row at this vocabulary)
    g = torch.Generator().manual_seed(block * 100 + blocks)
    x = torch.randn(rows, vocab, generator=g).to(torch.bfloat16)
    x[::3, 7] = 12.0                                      # confident rows
    cur = torch.randint(0, vocab - 1, (rows,), generator=g, dtype=torch.int32)
    cur[torch.rand(rows, generator=g) < 0.5] = vocab - 1
    x.view(blocks, block, vocab)[::2, :, 7] = 0.0         # blocks without a confident row: forced
    if block > 2:
        x.view(blocks, block, vocab)[0, 1:] = x[0]        # equal confidences: the lowest masked row
    ref = oracle.threshold_update(x, cur, vocab - 1, block, 0.9, 0.0, with_entropy=True)
    for gate in (None, 1, 0):
        kw = {} if gate is None else {"run_if_nonzero": torch.tensor([gate], dtype=torch.int32, device=DEV)}
        got = gpu.threshold_update(x.to(DEV), cur.to(DEV), vocab - 1, block, 0.9, 0.0, with_entropy=True, **kw)
        torch.cuda.synchronize()
        if gate == 0:
            assert torch.equal(got["new_tokens"].cpu(), cur) and not got["action"].any() and not got["block_changed"].any()
            assert int(got["changed_count"]) == 0
            continue
        act, want = got["action"].cpu().numpy().reshape(blocks, block), ref["action"].reshape(blocks, block)
        same = np.ones(blocks, dtype=bool)
        for i in range(blocks):                           # a forced row may be another within fp32 rounding of the best
            if (act[i] != want[i]).any():
                c = ref["conf"].reshape(blocks, block)[i]
                f, r = np.nonzero(act[i] == 2)[0], np.nonzero(want[i] == 2)[0]
                assert len(f) == len(r) == 1 and c[f[0]] >= c[r[0]] * (1 - 1e-5), f"block {i}"
                same[i] = False
        rows_same = np.repeat(same, block)
        assert np.array_equal(got["new_tokens"].cpu().numpy()[rows_same], ref["new_tokens"][rows_same])
        assert np.array_equal(got["block_changed"].cpu().numpy(), ref["block_changed"])
        if block > 2 and same[0] and (want[0] == 2).any():
            assert np.nonzero(act[0] == 2)[0][0] == np.nonzero(cur.numpy()[:block] == vocab - 1)[0][0]
        assert int(got["changed_count"]) == ref["changed_count"]


@pytest.mark.parametrize("block", [1, 2, 3, 16, 31, 32, 33, 63, 64, 65, 257])
@pytest.mark.parametrize("blocks", [1, 5, 64])
def test_tail_scores(gpu, block, blocks):
    e = torch.rand(blocks * block, generator=torch.Generator().manual_seed(block), dtype=torch.float32) * 9
    e[::4] = 3.25                                         # ties
    for rho in (0.01, 0.25, 1.0):
        got = gpu.tail_entropy_scores(e.to(DEV), block, rho).cpu()
        k = max(1, math.ceil(rho * block))
        top = e.view(blocks, block).double().sort(dim=1, descending=True).values[:, :k].mean(dim=1)
        # k fp32 additions of positive terms and a division
        assert torch.all((got.double() - top).abs() <= (k + 1) * 2.0 ** -24 * top), f"block {block} rho {rho}"
