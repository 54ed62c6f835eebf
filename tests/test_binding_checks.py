"""What the Python binding refuses before it calls the library: tensors that
are not on a GPU (whose addresses a kernel must never see), and, on the GPU,
every tensor argument of the attention with a wrong type, device, layout or
shape in turn (the binding tests the usual case in one condition, and names
what is wrong only when that fails)."""
import pytest
import torch

import paper_2607_22663_amd as mbe


def _attn_args(dev):
    q = torch.zeros(32, 8, 64, dtype=torch.bfloat16, device=dev)
    k = torch.zeros(6, 2, 16, 64, dtype=torch.bfloat16, device=dev)
    v = torch.zeros(6, 2, 64, 16, dtype=torch.bfloat16, device=dev)
    table = torch.arange(6, dtype=torch.int32, device=dev).view(1, 6)
    return [q, k, v, table, torch.full((1,), 64, dtype=torch.int32, device=dev),
            torch.full((1,), 32, dtype=torch.int32, device=dev)]


def test_host_tensors_are_refused():
    """On a machine with a GPU and without: the binding itself refuses them, by
    the stream it cannot get for them, before the library is called."""
    a = _attn_args("cpu")
    kw = dict(max_prefix_len=64)
    logits, cur = torch.zeros(32, 64, dtype=torch.bfloat16), torch.zeros(32, dtype=torch.int32)
    calls = [lambda: mbe.window_attention(*a, 32, max_window_len=32, **kw),
             lambda: mbe.block_diffusion_attention(*a[:5], 32, **kw),
             lambda: mbe.edit_select(logits, cur, 0.5),
             lambda: mbe.threshold_update(logits, cur, 63, 32, 0.5, 0.0),
             lambda: mbe.tail_entropy_scores(torch.zeros(32), 32, 0.5),
             lambda: mbe.select_start_block(torch.zeros(1, 4), torch.zeros(1, dtype=torch.int32), 2),
             lambda: mbe.refresh_blocks(torch.zeros(1, 4, dtype=torch.uint8)),
             lambda: mbe.kv_write(a[1], a[2], a[3], a[4], a[5], a[0][:, :2].contiguous(), a[0][:, :2].contiguous(),
                                  max_len=32)]
    reached = []

    class Lib:
        """The library, with calls that would launch recorded instead."""
        def __getattr__(self, name):
            f = getattr(real, name)
            return f if "workspace" in name or name == "mbe_last_error" else lambda *x: reached.append(name) or 0

    real, mbe._lib = mbe.load(), Lib()
    try:
        for call in calls:
            with pytest.raises((ValueError, RuntimeError, AssertionError)) as e:
                call()
            assert not isinstance(e.value, mbe.MbeError), e.value
    finally:
        mbe._lib = real
    assert not reached, reached


NAMES = ["q", "k_pages", "v_pages", "page_table", "prefix_lens", "window_lens", "out"]


@pytest.mark.gpu
@pytest.mark.parametrize("which", range(7))
@pytest.mark.parametrize("fault", ["type", "device", "strides", "dims", "none", "list"])
def test_each_argument_is_checked(gpu, which, fault):
    a = _attn_args("cuda:0") + [torch.zeros(32, 8, 64, dtype=torch.bfloat16, device="cuda:0")]
    t = a[which]
    if fault == "type":
        a[which] = t.to(torch.float32 if t.dtype == torch.bfloat16 else torch.int64)
    elif fault == "device":
        a[which] = t.cpu()
    elif fault == "strides":
        if t.numel() == 1:
            pytest.skip("one element is always contiguous")
        a[which] = torch.stack([t, t], dim=-1)[..., 0]
        assert not a[which].is_contiguous()
    elif fault == "dims":
        a[which] = t.unsqueeze(0)
    elif fault == "none":
        if NAMES[which] == "out":
            pytest.skip("out may be left out")
        a[which] = None
    else:
        a[which] = [1, 2, 3]
    with pytest.raises((TypeError, ValueError, AttributeError)):
        gpu.window_attention(*a[:6], 32, out=a[6], max_prefix_len=64, max_window_len=32)


@pytest.mark.gpu
def test_usual_call_runs(gpu):
    a = _attn_args("cuda:0")
    out = gpu.window_attention(*a, 32, max_prefix_len=64, max_window_len=32)
    torch.cuda.synchronize()
    assert out.shape == a[0].shape and bool((out == 0).all())


@pytest.mark.gpu
def test_vocab_zero_raises(gpu):
    logits = torch.zeros(32, 64, dtype=torch.bfloat16, device="cuda:0")
    cur = torch.zeros(32, dtype=torch.int32, device="cuda:0")
    with pytest.raises(gpu.MbeError, match="vocab must be >= 1"):
        gpu.threshold_update(logits, cur, 63, 32, 0.5, 0.0, vocab=0)
    with pytest.raises(gpu.MbeError, match="vocab must be >= 1"):
        gpu.edit_select(logits, cur, 0.5, vocab=0)
