"""Rows that start off the 16-byte grid, through edit selection and the update.

A row's first logits up to the next multiple of 16 bytes (its head) are read
one per thread, everything after them in whole 16-byte vectors.  Every start
offset 0..7 (elements past an aligned address, stride odd so that the offset
changes from row to row) at vocabularies around the head (1..17), around one
iteration of a workgroup (4096 logits) and around two chunks, with the
maximum planted in the head, right after it, at the row's end, and tied
between the head and the rest (the lowest index wins).  Logits outside the
vocabulary hold +inf, so a read past either end of a row shows."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _rows(vocab, seed):
    rng = np.random.default_rng(seed)
    rows = 32
    stride = vocab + 1 + vocab % 2 * 2 + 8 * int(rng.integers(0, 2))
    stride += 1 - stride % 2                                     # odd: offsets 0..7 all occur
    x = rng.normal(0.0, 3.0, size=(rows, vocab)).astype(np.float32)
    for r in range(rows):
        top = x[r].max() + 4.0
        kind = r % 5
        if kind == 0:
            x[r, 0] = top
        elif kind == 1:
            x[r, min(vocab - 1, 7 + r % 3)] = top
        elif kind == 2:
            x[r, vocab - 1] = top
        elif kind == 3:
            x[r, min(vocab - 1, int(rng.integers(0, 8)))] = top
            x[r, rng.integers(0, vocab, size=3)] = top           # ties, the lowest index wins
        if vocab > 2 and r % 4 == 1:
            x[r, rng.integers(0, vocab)] = -np.inf
            x[r, vocab // 2] = max(x[r, vocab // 2], 0.0)
    return torch.from_numpy(x).to(torch.bfloat16), stride


@pytest.mark.parametrize("vocab", [1, 2, 7, 8, 9, 15, 16, 17, 4088, 4095, 4096, 4097, 4104, 8191, 8192, 8200, 12289, 50001])
def test_rows_off_the_16_byte_grid(gpu, vocab):
    x, stride = _rows(vocab, vocab)
    rows = x.shape[0]
    buf = torch.full((8 + rows * stride + 8,), float("inf"), dtype=torch.bfloat16)
    cur = torch.from_numpy(np.random.default_rng(1).integers(0, vocab, size=rows).astype(np.int32))
    ref_n, ref_c, ref_ch = oracle.edit_select(x, cur, 0.0)
    ref_u = oracle.threshold_update(x, cur, vocab, 8, 0.5, 0.0, with_entropy=True)
    for off in range(8):
        full = buf.clone()
        view = full[off:off + rows * stride].view(rows, stride)
        view[:, :vocab] = x
        d = full.to(DEV)[off:off + rows * stride].view(rows, stride)
        n, c, ch = gpu.edit_select(d, cur.to(DEV), 0.0, vocab=vocab)
        u = gpu.threshold_update(d, cur.to(DEV), vocab, 8, 0.5, 0.0, vocab=vocab, with_entropy=True)
        torch.cuda.synchronize()
        assert np.array_equal(n.cpu().numpy(), ref_n), (vocab, off)
        assert np.array_equal(ch.cpu().numpy(), ref_ch), (vocab, off)
        # fp32 sums of at most 50001 terms in a tree: within 1e-6 relative, as everywhere in this suite
        assert np.max(np.abs(c.cpu().numpy() - ref_c) / ref_c) <= 1e-6, (vocab, off)
        assert np.array_equal(u["new_tokens"].cpu().numpy(), ref_u["new_tokens"]), (vocab, off)
        # entropy = ln 2 (log2 s - t / s): absolute error of a few fp32 ulps of log2 s <= 16
        assert np.max(np.abs(u["entropy"].cpu().numpy() - ref_u["entropy"])) <= 1e-5, (vocab, off)


LOWEST = float(torch.finfo(torch.bfloat16).min)


@pytest.mark.parametrize("mask", [LOWEST, -float("inf")])
@pytest.mark.parametrize("vocab", [9, 17, 1000, 4096, 4103, 5000, 9001, 50001])
def test_masked_logits(gpu, vocab, mask):
    """Logits masked with the type's lowest value or -inf: the first or the last
    few (a row's head and tail), a leading or trailing range, every second one, and all
    but one.  The masked ones have probability 0 in fp64 too (the rest is
    within 60 of the maximum), so confidences and entropies are those of the
    rest."""
    rng = np.random.default_rng(vocab)
    rows, stride = 32, vocab + 1 + vocab % 2
    x = rng.normal(0.0, 3.0, size=(rows, vocab)).astype(np.float32)
    for r in range(rows):
        n = vocab - 1
        keep = x[r].copy()
        kind = r % 8
        if kind == 0:
            x[r, :1 + r % 7] = mask
        elif kind == 1:
            x[r, -(1 + r % 7):] = mask
        elif kind == 2:
            x[r, :n // 2 + 1] = mask
        elif kind == 3:
            x[r, n // 2 + 1:] = mask
        elif kind == 4:
            x[r, r // 8 % 2::2] = mask
        elif kind == 5:
            x[r] = mask
        elif kind == 6:
            x[r, : min(n, 8 - r // 8)] = mask
            x[r, -min(n, 600):] = mask
        at = [n, 0, n, 0, n - (n + r // 8 + 1) % 2, int(rng.integers(0, vocab)), n // 2, n][kind]
        x[r, at] = keep[at] if kind != 5 else 1.5            # one at least is never masked
    x = torch.from_numpy(x).to(torch.bfloat16)
    cur = torch.from_numpy(rng.integers(0, vocab, size=rows).astype(np.int32))
    ref_n, ref_c, ref_ch = oracle.edit_select(x, cur, 0.0)
    xd = x.double().numpy()
    p = np.exp(xd - xd.max(axis=1, keepdims=True))
    p /= p.sum(axis=1, keepdims=True)
    ref_h = -np.sum(np.where(p > 0, p * np.log(np.where(p > 0, p, 1.0)), 0.0), axis=1)
    for off in range(8):
        d = torch.zeros(8 + rows * stride + 8, dtype=torch.bfloat16)
        d[off:off + rows * stride].view(rows, stride)[:, :vocab] = x
        d = d.to(DEV)[off:off + rows * stride].view(rows, stride)
        n, c, ch = gpu.edit_select(d, cur.to(DEV), 0.0, vocab=vocab)
        u = gpu.threshold_update(d, cur.to(DEV), vocab, 8, 0.5, 0.0, vocab=vocab, with_entropy=True)
        torch.cuda.synchronize()
        assert np.array_equal(n.cpu().numpy(), ref_n) and np.array_equal(ch.cpu().numpy(), ref_ch), off
        for got in (c, u["conf"]):
            assert np.max(np.abs(got.cpu().numpy() - ref_c) / ref_c) <= 1e-6, off
        assert np.max(np.abs(u["entropy"].cpu().numpy() - ref_h)) <= 1e-5, off


@pytest.mark.parametrize("vocab", [2, 9, 17, 1000, 4103, 5000, 9001, 50001])
def test_a_nan_logit_keeps_the_token(gpu, vocab):
    """One NaN in a row of finite logits, at either end or anywhere: without
    entropies its confidence is NaN, which clears no threshold, whichever thread
    and iteration meets it."""
    rng = np.random.default_rng(vocab)
    rows, stride = 32, vocab + 1 + vocab % 2
    x = rng.normal(0.0, 3.0, size=(rows, vocab)).astype(np.float32)
    ends = [c % vocab for e in range(9) for c in (e, vocab - 1 - e)]
    for r in range(rows):
        x[r, ends[r] if r < len(ends) else rng.integers(0, vocab)] = np.nan
    x = torch.from_numpy(x).to(torch.bfloat16)
    cur = torch.full((rows,), vocab, dtype=torch.int32, device=DEV)      # differs from every prediction
    for off in range(8):
        d = torch.zeros(8 + rows * stride + 8, dtype=torch.bfloat16)
        d[off:off + rows * stride].view(rows, stride)[:, :vocab] = x
        d = d.to(DEV)[off:off + rows * stride].view(rows, stride)
        n, c, ch = gpu.edit_select(d, cur, 0.0, vocab=vocab)
        torch.cuda.synchronize()
        assert bool(torch.isnan(c).all()) and bool((n == cur).all()) and not bool(ch.any()), off
