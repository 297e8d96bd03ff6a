"""The sweeps read x and dy and write dx where the caller has them, without copies, unless that is not the same as copying first:
buffers that overlap, that are not 16-byte aligned or lie in host memory give the same bits as buffers of their own, and the
checkpoints hold x and y."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2106_02679_amd import binding as B
from gpu_helpers import TORCH_DTYPE

SIZES = [(B.LGA_BF16, 128, 2, 512), (B.LGA_BF16, 1536, 12, 6144), (B.LGA_FP32, 64, 4, 256), (B.LGA_FP32, 30, 3, 70)]      # fp32 rows of 30: no 16-byte pieces


def make(dt, d, heads, ff, layers, group):
    cfg = B.make_config(layers, d, heads, ff, 40, 1, 4, dt, group=group, retain_grads=1)
    params = np.random.default_rng(1).standard_normal(layers * B.params_per_layer(cfg)).astype(np.float32) * 0.02
    return B.Stack(cfg, params), 4 * 40 * d


@pytest.mark.parametrize("dt,d,heads,ff", SIZES, ids=["bf16_128", "bf16_1536", "fp32_64", "fp32_30"])
@pytest.mark.parametrize("layers,group", [(1, 1), (2, 2)])
def test_forward_buffers_that_overlap_or_are_misaligned(dt, d, heads, ff, layers, group):
    st, n = make(dt, d, heads, ff, layers, group)
    row, shift = 40 * d, 4
    x0 = torch.randn(n, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3)).to(TORCH_DTYPE[dt])

    def run(x_at, y_at, per_layer=False):
        buf = torch.full((3 * n + 64,), float("nan"), device="cuda", dtype=x0.dtype)
        x, y = buf[x_at:x_at + n], buf[y_at:y_at + n]
        x.copy_(x0)
        if per_layer:
            for l in range(layers):
                st.forward_layer(l, (x if l == 0 else y).data_ptr(), y.data_ptr())
        else:
            st.forward_layered(x.data_ptr(), y.data_ptr())
        torch.cuda.synchronize()
        kept = [B.read_device(st.checkpoint(b)[0], n, "float32" if dt == B.LGA_FP32 else "uint16") for b in ([0] if per_layer else [0, layers])]
        return y.clone(), kept

    try:
        ref, kept = run(0, 2 * n)
        view = lambda t: (t if dt == B.LGA_FP32 else t.view(torch.int16)).cpu().numpy().view("float32" if dt == B.LGA_FP32 else "uint16")
        assert torch.isfinite(ref.float()).all()
        assert np.array_equal(kept[0], view(x0)) and np.array_equal(kept[1], view(ref))
        for args in ((0, 0), (0, row), (row, 0), (shift // 2, 2 * n), (0, 2 * n + shift // 2), (0, 2 * n, True), (0, 0, True), (row, 0, True), (0, row, True)):
            y, k = run(*args)
            assert torch.equal(y, ref) and np.array_equal(k[0], kept[0]), args
            assert len(k) == 1 or np.array_equal(k[1], kept[1]), args
        pinned = torch.empty(2, n, dtype=x0.dtype, pin_memory=True)
        pinned[0].copy_(x0)
        st.forward_layered(pinned[0].data_ptr(), pinned[1].data_ptr())
        torch.cuda.synchronize()
        assert torch.equal(pinned[1], ref.cpu())
    finally:
        st.close()


@pytest.mark.parametrize("dt,d,heads,ff", SIZES, ids=["bf16_128", "bf16_1536", "fp32_64", "fp32_30"])
@pytest.mark.parametrize("layers", [1, 2])
def test_micro_batch_major_buffers_that_overlap(dt, d, heads, ff, layers):
    st, n = make(dt, d, heads, ff, layers, 1)
    row = 40 * d
    gen = torch.Generator(device="cuda").manual_seed(4)
    x0, g0 = (torch.randn(n, device="cuda", generator=gen).to(TORCH_DTYPE[dt]) for _ in range(2))

    def run(x_at, g_at, y_at, dx_at):
        buf = torch.full((8 * n,), float("nan"), device="cuda", dtype=x0.dtype)
        x, g, y, dx = (buf[a:a + n] for a in (x_at, g_at, y_at, dx_at))
        x.copy_(x0)
        g.copy_(g0)
        st.step_mbmajor(x.data_ptr(), g.data_ptr(), y.data_ptr(), dx.data_ptr(), None)
        torch.cuda.synchronize()
        return [y.clone(), dx.clone()] + [torch.from_numpy(B.read_device(*st.grads(l), "float32")) for l in range(layers)]

    try:
        ref = run(0, 2 * n, 4 * n, 6 * n)
        assert torch.isfinite(ref[1].float()).all()
        for args in ((0, 2 * n, 0, 2 * n), (0, 2 * n, 0, 6 * n), (0, 2 * n, 4 * n, 2 * n + row), (0, 2 * n, row, 6 * n), (row, 3 * n, 6 * n, 0), (0, 2 * n, 4 * n + 2, 6 * n)):
            for got, want in zip(run(*args), ref):
                assert torch.equal(got, want), args
    finally:
        st.close()


@pytest.mark.parametrize("layers", [1, 2])
@pytest.mark.parametrize("before", [0, 1, 3])
def test_where_y_and_dx_overlap_dx_is_what_stays(layers, before):
    """Micro-batch order: y is complete before dx is, so that a program with no use for y may give both one buffer.  before: rows that y begins
    ahead of dx, which keep y's values."""
    st, n = make(B.LGA_BF16, 128, 2, 512, layers, 1)
    row = 40 * 128
    gen = torch.Generator(device="cuda").manual_seed(5)
    x, g = (torch.randn(n, device="cuda", generator=gen).bfloat16() for _ in range(2))
    try:
        y, dx = torch.empty_like(x), torch.empty_like(x)
        st.step_mbmajor(x.data_ptr(), g.data_ptr(), y.data_ptr(), dx.data_ptr(), None)
        buf = torch.full((2 * n,), float("nan"), device="cuda", dtype=x.dtype)
        st.step_mbmajor(x.data_ptr(), g.data_ptr(), buf.data_ptr(), buf[before * row:].data_ptr(), None)
        torch.cuda.synchronize()
        assert torch.equal(buf[before * row:before * row + n], dx) and torch.equal(buf[:before * row], y[:before * row])
    finally:
        st.close()


@pytest.mark.parametrize("which", ["x", "x_in", "dy", "layer_dy", "dx", "mb_x", "mb_dy", "mb_dx"])
def test_a_buffer_shorter_than_the_activations_is_refused(which):
    """16 bytes short, in an allocation of its own whose last page holds those 16 bytes all the same: the call reports an error, as the copy
    that the sweeps once made of it did, and the stack goes on working."""
    import ctypes as C
    hip = C.CDLL("libamdhip64.so.7")
    st, n = make(B.LGA_BF16, 128, 2, 512, 1, 1)
    short, p = 2 * n - 16, C.c_void_p()
    assert 0 < short % 4096 <= 4096 - 16                             # (16 more bytes do not reach another page)
    assert hip.hipMalloc(C.byref(p), C.c_size_t(short)) == 0
    x, g, y, dx = (torch.randn(n, device="cuda").bfloat16() for _ in range(4))
    own = {k: t.data_ptr() for k, t in (("x", x), ("g", g), ("y", y), ("dx", dx))}
    calls = {"x": lambda a, _: st.forward_layered(a, own["y"]),
             "x_in": lambda a, _: st.forward_layer(0, a, own["y"]),
             "dy": lambda a, _: st.backward_layered(a, own["dx"], None),
             "layer_dy": lambda a, _: st.backward_layer(0, a, own["dx"], None),
             "dx": lambda _, b: st.backward_layered(own["g"], b, None),
             "mb_x": lambda a, _: st.step_mbmajor(a, own["g"], own["y"], own["dx"], None),
             "mb_dy": lambda a, _: st.step_mbmajor(own["x"], a, own["y"], own["dx"], None),
             "mb_dx": lambda _, b: st.step_mbmajor(own["x"], own["g"], own["y"], b, None)}
    try:
        st.forward_layered(own["x"], own["y"])
        torch.cuda.synchronize()
        with pytest.raises(B.LgaError) as e:
            calls[which](p.value, p.value)
        assert e.value.code == B.LGA_ERR_HIP
        torch.cuda.synchronize()
        st.forward_layered(own["x"], own["y"])
        st.backward_layered(own["g"], own["dx"], None)
        torch.cuda.synchronize()
        assert torch.isfinite(dx.float()).all()
    finally:
        torch.cuda.synchronize()
        st.close()
        assert hip.hipFree(p) == 0
