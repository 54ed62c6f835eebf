"""Edit selection and the update on both sides of their launch rules: rows
cut into chunks or not (the vocabulary where the rule turns, for several row
counts), 512 threads per row below 512 rows and 256 from there, and the update's
merge of 1 to 64+ chunks per row inside its per-block step, for blocks of one
row, of a ragged size and of all rows; against the oracle, in-place tokens
included.  A subset of the rows is compared where the oracle would be slow."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _logits(rows, vocab, seed):
    g = torch.Generator(DEV).manual_seed(seed)
    x = torch.empty(rows, vocab, dtype=torch.bfloat16, device=DEV).normal_(0.0, 3.0, generator=g)
    col = torch.randint(0, vocab, (rows,), generator=g, device=DEV)
    x[torch.arange(rows, device=DEV), col] = 16.0           # exact in bf16, above every other
    # some rows tied with an earlier column (another chunk)
    tie = torch.arange(0, rows, 3, device=DEV)
    x[tie, col[tie] // 2] = 16.0
    cur = torch.randint(0, vocab, (rows,), generator=g, device=DEV, dtype=torch.int32)
    return x, cur


# (rows, vocab, whether its rows are cut): both sides of the turns of the rule,
# at 80000 logits for the fewest rows, 100000 at 128 and 288, 200000 at 160
@pytest.mark.parametrize("rows,vocab,cut", [
    (1, 80000, False), (1, 80001, True), (1, 4096, False), (1, 4097, False), (3, 200003, True),
    (64, 80000, False), (64, 80001, True), (128, 100000, False), (128, 100001, True), (160, 200000, False),
    (160, 200001, True), (176, 131072, False), (256, 131073, False), (257, 80000, False), (288, 100000, False),
    (288, 100001, True), (384, 131072, True), (385, 131072, False), (511, 20000, False), (512, 20000, False),
    (513, 8191, False)])
def test_edit_select_plans(gpu, rows, vocab, cut):
    assert (gpu.load().mbe_edit_select_workspace_size(rows, vocab) > 0) == cut
    x, cur = _logits(rows, vocab, rows + vocab)
    n, c, ch = gpu.edit_select(x, cur, 0.5)
    torch.cuda.synchronize()
    pick = np.unique(np.linspace(0, rows - 1, min(rows, 24)).astype(int))
    rn, rc, rch = oracle.edit_select(x[pick].cpu(), cur[pick].cpu(), 0.5)
    assert np.array_equal(n[pick].cpu().numpy(), rn) and np.array_equal(ch[pick].cpu().numpy(), rch)
    assert np.max(np.abs(c[pick].cpu().numpy() - rc) / rc) <= 1e-6


@pytest.mark.parametrize("rows,vocab,block", [(1, 300000, 1), (2, 131072, 2), (7, 262144, 7), (30, 65537, 10), (96, 131072, 96),
                                              (256, 131072, 256), (500, 16384, 250), (512, 16384, 512), (48, 9000, 3)])
@pytest.mark.parametrize("entropy", [True, False])
def test_update_merges_chunks(gpu, rows, vocab, block, entropy):
    x, cur = _logits(rows, vocab, rows * 7 + vocab)
    cur[torch.arange(0, rows, 2, device=DEV)] = vocab         # masked rows
    ref = None
    if rows * vocab <= 20_000_000:
        ref = oracle.threshold_update(x.cpu(), cur.cpu(), vocab, block, 0.5, 0.0, with_entropy=entropy)
    out = gpu.threshold_update(x, cur, vocab, block, 0.5, 0.0, with_entropy=entropy)
    tokens = cur.clone()
    same = {k: torch.empty_like(v) for k, v in out.items()}
    same["new_tokens"] = tokens                               # in place
    gpu.threshold_update(x, tokens, vocab, block, 0.5, 0.0, out=same)
    torch.cuda.synchronize()
    for k in out:
        assert torch.equal(out[k], same[k]), f"{k}: in place differs"
    if ref is None:
        pick = np.unique(np.linspace(0, rows - 1, 12).astype(int))
        p, c = oracle.update.prediction(x[pick].cpu())
        got = out["new_tokens"][pick].cpu().numpy()
        act = out["action"][pick].cpu().numpy()
        assert np.array_equal(got[act != 0], p[act != 0])
        assert np.max(np.abs(out["conf"][pick].cpu().numpy() - c) / c) <= 1e-6
        return
    for k in ("new_tokens", "action", "block_changed"):
        assert np.array_equal(out[k].cpu().numpy().astype(np.int64), np.asarray(ref[k]).astype(np.int64)), k
    assert int(out["changed_count"][0]) == ref["changed_count"]
    assert np.max(np.abs(out["conf"].cpu().numpy() - ref["conf"]) / ref["conf"]) <= 1e-6
    if entropy:
        assert np.max(np.abs(out["entropy"].cpu().numpy() - ref["entropy"])) <= 1e-5


@pytest.mark.parametrize("vocab", [1, 9, 4095, 4096, 4097, 8192, 12300, 40961])
@pytest.mark.parametrize("rows", [512, 528, 640, 1408])
def test_one_or_two_iterations_in_flight(gpu, rows, vocab):
    """Both forms of the row loop, on either side of the rows where one takes
    over from the other (513 with entropies, 640 without, 1408): no whole
    iteration (4096 logits a workgroup), whole ones only, and a remainder, with
    rows on and off the 16-byte grid."""
    for stride in ((vocab + 7) // 8 * 8, vocab + 1 + vocab % 2):
        x = torch.full((rows, stride), float("inf"), dtype=torch.bfloat16, device=DEV)
        x[:, :vocab], cur = _logits(rows, vocab, rows + vocab)
        n, c, ch = gpu.edit_select(x, cur, 0.5, vocab=vocab)
        u = gpu.threshold_update(x, cur, vocab, 16, 0.5, 0.0, vocab=vocab, with_entropy=True)
        torch.cuda.synchronize()
        pick = np.unique(np.linspace(0, rows - 1, 24).astype(int))
        xp = x[pick, :vocab].cpu()
        rn, rc, rch = oracle.edit_select(xp, cur[pick].cpu(), 0.5)
        assert np.array_equal(n[pick].cpu().numpy(), rn) and np.array_equal(ch[pick].cpu().numpy(), rch)
        for got in (c, u["conf"]):
            assert np.max(np.abs(got[pick].cpu().numpy() - rc) / rc) <= 1e-6
        assert np.max(np.abs(u["entropy"][pick].cpu().numpy() - oracle.entropy.row_entropy(xp))) <= 1e-5
