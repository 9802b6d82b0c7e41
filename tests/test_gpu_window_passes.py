"""The window passes at the edges of their tasks, against the CPU oracle: every pass order (which lines of the far
faces a finest-level pass leaves out follows from it), fields that end on, one short of and one past a window, and
values that send a task down its rare branches (outliers, the FP64 bound test, predictions past the largest float)."""
import itertools

import numpy as np
import pytest

import oracle as O
import paper_2312_05492_amd as szi
from paper_2312_05492_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    O.build(force=False)
    c = szi.Context(0)
    yield c
    c.close()


def check(ctx, x, **kw):
    import torch
    print("\n[passes] %s %s" % (x.shape, kw), flush=True)
    ref = O.compress(x, O.Params(shape=x.shape, **kw))
    res = ctx.compress(torch.from_numpy(np.ascontiguousarray(x)).cuda(), **kw)
    try:
        assert np.array_equal(res.read(szi.SEC_CODES), ref.codes.ravel())
        assert res.blob() == ref.blob()
        y = ctx.decompress(res).cpu().numpy()
        assert np.array_equal(y.view(np.uint32), ref.recon.view(np.uint32))
    finally:
        res.free()


@pytest.mark.parametrize("order", list(itertools.permutations(range(3))))
@pytest.mark.parametrize("shape", [(16, 16, 64), (17, 9, 65), (18, 15, 63)])
def test_orders_3d(ctx, order, shape):
    check(ctx, synth.spectral_field(shape, seed=101), order=order, interp=(2, 1, 2), eb=1e-4)


@pytest.mark.parametrize("order", [(0, 1), (1, 0)])
@pytest.mark.parametrize("shape", [(32, 128), (33, 129), (31, 130)])
def test_orders_2d(ctx, order, shape):
    check(ctx, synth.spectral_field(shape, seed=102), order=order, interp=(1, 2), eb=1e-4)


@pytest.mark.parametrize("shape", [(20, 30, 70), (50, 140)])
def test_rare_branches(ctx, shape):
    rng = np.random.default_rng(103)
    x = synth.spectral_field(shape, seed=103)
    # spikes: scattered outliers; a bound of a few ulps of the offset field: differences that round to the bound
    check(ctx, np.where(rng.random(shape) < 0.01, x + np.float32(1e3), x).astype(np.float32), eb=1e-3, eb_mode=0)
    check(ctx, x + np.float32(1000.0), eb=2.0 ** -12, eb_mode=0, interp=(2,) * len(shape))
    # predictions that overflow
    big = np.where(rng.random(shape) < 0.5, np.float32(3e38), np.float32(-3e38)).astype(np.float32)
    check(ctx, big, eb=1e30, eb_mode=0, interp=(2,) * len(shape))


@pytest.mark.parametrize("interp", [0, 1, 2])
@pytest.mark.parametrize("n", [2, 31, 32, 33, 65, 511, 512, 513, 1025, 1537, 1985, 2016, 2017, 2047, 4096, 4097, 6143,
                               10240, 8 * 2048 * 4 + 7])
def test_line_sizes(ctx, n, interp):
    check(ctx, synth.spectral_field((n,), seed=104), interp=(interp,), eb=1e-3)


def test_line_rare_branches(ctx):
    rng = np.random.default_rng(105)
    x = synth.spectral_field((9000,), seed=105)
    check(ctx, np.where(rng.random(9000) < 0.01, x + np.float32(1e3), x).astype(np.float32), eb=1e-3, eb_mode=0)
    check(ctx, x + np.float32(1000.0), eb=2.0 ** -12, eb_mode=0, interp=(2,))
    big = np.where(rng.random(9000) < 0.5, np.float32(3e38), np.float32(-3e38)).astype(np.float32)
    check(ctx, big, eb=1e30, eb_mode=0, interp=(2,))


# (shape, stride, window): block sizes on both sides of the kernels' LDS sizes (1152, 2816 and 4096 words), long and
# thin windows, ragged fields whose last windows hold a single plane
GENERAL = [((33, 34, 25), 8, (16, 16, 8)), ((17, 40, 50), 8, (8, 8, 24)), ((9, 25, 98), 8, (8, 8, 48)),
           ((20, 33, 35), 4, (12, 16, 16)), ((13, 14, 15), 2, (2, 2, 2)), ((40, 41, 43), 4, (8, 8, 32)),
           ((33, 65), 32, (32, 32)), ((34, 130), 16, (32, 96)), ((70, 45), 4, (60, 4)), ((2100,), 8, (1024,)),
           ((1030,), 2, (2,)), ((5000,), 256, (768,))]


@pytest.mark.parametrize("shape,stride,window", GENERAL)
@pytest.mark.parametrize("interp", [0, 1, 2])
def test_other_windows(ctx, shape, stride, window, interp):
    x = synth.spectral_field(shape, seed=106)
    check(ctx, x, S=stride, window=window, interp=(interp,) * len(shape), eb=1e-3)


def test_other_window_orders_and_rare_branches(ctx):
    x = synth.spectral_field((20, 35, 30), seed=107)
    for order in itertools.permutations(range(3)):
        check(ctx, x, S=8, window=(16, 16, 8), order=order, interp=(2, 1, 0), eb=1e-4)
    rng = np.random.default_rng(108)
    check(ctx, np.where(rng.random(x.shape) < 0.01, x + np.float32(1e3), x).astype(np.float32), S=4, eb=1e-3, eb_mode=0)
    check(ctx, x + np.float32(1000.0), S=4, eb=2.0 ** -12, eb_mode=0, interp=(2, 2, 2))


def off_alignment(x, shift):
    """x on the GPU, shift floats past a 16-byte boundary, and its buffer with guard values around it."""
    import torch
    buf = torch.full((x.size + 8,), -7.0, dtype=torch.float32, device="cuda")
    view = buf[4 + shift:4 + shift + x.size].view(x.shape)
    view.copy_(torch.from_numpy(np.ascontiguousarray(x)))
    return view, buf


@pytest.mark.parametrize("shift", [1, 2, 3])
@pytest.mark.parametrize("shape,stride,window", [((33, 34, 25), 8, (16, 16, 8)), ((34, 130), 16, (32, 96)),
                                                 ((5000,), 256, (768,))])
def test_other_windows_off_alignment(ctx, shape, stride, window, shift):
    x = synth.spectral_field(shape, seed=109)
    kw = dict(S=stride, window=window, eb=1e-3)
    ref = O.compress(x, O.Params(shape=shape, **kw))
    print("\n[passes] %s off by %d" % (shape, shift), flush=True)
    res = ctx.compress(off_alignment(x, shift)[0], **kw)
    assert res.blob() == ref.blob()
    out, buf = off_alignment(np.zeros_like(x), shift)
    ctx.decompress(res, out)
    assert np.array_equal(out.cpu().numpy().view(np.uint32), ref.recon.view(np.uint32))
    y = buf.cpu().numpy()
    assert (y[:4 + shift] == -7.0).all() and (y[4 + shift + x.size:] == -7.0).all()   # nothing outside
    res.free()


def test_lines_of_a_batch_on_and_off_alignment(ctx):
    # a workgroup's windows come from fields on and one to three floats off 16 bytes by turns: loaded ahead or not
    xs = [synth.spectral_field((n,), seed=110 + i) for i, n in
          enumerate([9000, 4096, 70001, 2047, 2048, 2049, 30000, 8192, 6143, 12288, 5, 20480])]
    kws = [dict(eb=1e-3)] * len(xs)
    refs = [O.compress(x, O.Params(shape=x.shape, **kw)) for x, kw in zip(xs, kws)]
    print("\n[passes] lines on and off alignment", flush=True)
    for turn in range(2):
        res = ctx.compress_batch([off_alignment(x, (i + turn) % 4)[0] for i, x in enumerate(xs)], kws)
        for r, ref in zip(res, refs):
            assert r.blob() == ref.blob()
        outs = [off_alignment(np.zeros_like(x), (3 * i + turn) % 4) for i, x in enumerate(xs)]
        ctx.decompress_batch(res, [o for o, _ in outs])
        for i, ((o, buf), ref) in enumerate(zip(outs, refs)):
            assert np.array_equal(o.cpu().numpy().view(np.uint32), ref.recon.view(np.uint32)), i
            s, y = 4 + (3 * i + turn) % 4, buf.cpu().numpy()
            assert (y[:s] == -7.0).all() and (y[s + xs[i].size:] == -7.0).all()
        for r in res:
            r.free()
