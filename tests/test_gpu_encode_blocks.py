"""The Huffman encode's block sizes and sums against the CPU oracle: chunk counts on both sides of each number of
chunks per workgroup (4, 8, 16, 32), fields that end inside a block and inside a long sum, fields whose zero words
are elided and ones that keep them, batches whose fields' sums lie side by side, and more blocks than the short
sums serve."""
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


def smooth(n):
    """A slow wave with a quiet stretch: most Huffman words are zero."""
    t = np.arange(n, dtype=np.float64)
    return (np.sin(t * 1e-4) * (1.0 + 0.5 * np.sin(t * 3e-7))).astype(np.float32)


def rough(n):
    return np.random.default_rng(n).normal(size=n).astype(np.float32)


def check(ctx, x, **kw):
    import torch
    print("\n[encode] %s %s" % (x.shape, kw), flush=True)
    ref = O.compress(x, O.Params(shape=x.shape, **kw))
    res = ctx.compress(torch.from_numpy(x).cuda(), **kw)
    try:
        assert np.array_equal(res.read(szi.SEC_WORDS), ref.words)
        assert np.array_equal(res.read(szi.SEC_OUTLIER_IDX), ref.outlier_idx)
        blob = res.blob()
        assert blob == ref.blob()
        y = ctx.decompress(res).cpu().numpy()
        assert np.array_equal(y.view(np.uint32), ref.recon.view(np.uint32))
        # the elided words are restored from the blob
        up = ctx.upload(blob)
        assert np.array_equal(up.read(szi.SEC_WORDS), ref.words)
        up.free()
        return blob
    finally:
        res.free()


@pytest.mark.parametrize("chunks", [4, 5, 64 * 4, 64 * 4 + 1, 16383, 16385, 32769, 65535, 65537])
@pytest.mark.parametrize("gen", [smooth, rough])
def test_block_sizes(ctx, chunks, gen):
    check(ctx, gen(chunks * 256 - 77), chunk=256, eb=1e-2 if gen is rough else 1e-3)


def test_batch_of_block_counts(ctx):
    # fields of one to a few hundred blocks, elided and not, two chunk sizes
    import torch
    sizes = [(300, smooth, 256), (70000, rough, 256), (65536 * 4, smooth, 256), (1, rough, 256), (200000, smooth, 1024),
             (65536 * 16 + 5, rough, 1024), (900000, smooth, 256), (5000, smooth, 1024)]
    xs = [g(n) for n, g, _ in sizes]
    params = [dict(chunk=c, eb=1e-3) for _, _, c in sizes]
    refs = [O.compress(x, O.Params(shape=x.shape, **p)) for x, p in zip(xs, params)]
    for rep in range(2):
        print("\n[encode] batch, pass %d" % rep, flush=True)
        outs = ctx.compress_batch([torch.from_numpy(x).cuda() for x in xs], params)
        for r, ref in zip(outs, refs):
            assert r.blob() == ref.blob()
            r.free()


def test_given_code_with_many_outliers_runs_the_encode_again(ctx):
    import torch
    x = rough(300000)
    kw = dict(eb=1e-30, eb_mode=0)
    ref = O.compress(x, O.Params(shape=x.shape, **kw))
    book = szi.code_lengths(ref.hist)
    want = O.compress(x, O.Params(shape=x.shape, **kw), lengths=book)
    print("\n[encode] again", flush=True)
    res = ctx.compress_with_code(torch.from_numpy(x).cuda(), book, **kw)
    assert res.blob() == want.blob()
    res.free()


@pytest.mark.parametrize("chunk", [256, 512, 1024, 2048])
@pytest.mark.parametrize("every", [0, 1, 3, 50, 3000])
def test_outlier_lists(ctx, chunk, every):
    # a chunk's outliers: all its symbols (every 0: a bound of zero), most, one in 50, one in several chunks; the last
    # chunk ends inside a lane's symbols
    x = rough(chunk * 41 + 5)
    if every > 1:
        x[np.arange(x.size) % every != 0] = 0.0
    check(ctx, x, chunk=chunk, eb=0.0 if every == 0 else 1e-6, eb_mode=0)


def test_more_blocks_than_short_sums(ctx):
    # 2^27 points in chunks of 256: more than 16384 blocks of 32 chunks
    x = smooth(2 ** 27 + 12345)
    blob = check(ctx, x, chunk=256, eb=1e-4)
    assert blob[124] & 1   # elided


@pytest.mark.parametrize("given", [False, True])
def test_long_sums_of_a_batch(ctx, given):
    # more than 16384 blocks over fields of 0 to about 9500, whose long sums (over 256 blocks, scanned) lie side by
    # side: a field of none, of one less a block, of exactly one and of many, elided and not
    import torch
    block = 32 * 256
    sizes = [(100, rough), (255 * block, smooth), (256 * block, smooth), (256 * block + 1, rough), (5, smooth),
             (9500 * block - 3, smooth), (6500 * block, rough)]
    xs = [g(n) for n, g in sizes]
    p = dict(chunk=256, eb=1e-3)
    refs = [O.compress(x, O.Params(shape=x.shape, **p)) for x in xs]
    gs = [torch.from_numpy(x).cuda() for x in xs]
    print("\n[encode] batch of long sums, given %s" % given, flush=True)
    if given:
        books = [szi.code_lengths(r.hist) for r in refs]
        refs = [O.compress(x, O.Params(shape=x.shape, **p), lengths=b) for x, b in zip(xs, books)]
        outs = ctx.compress_batch_with_code(gs, books, [p] * len(xs))
    else:
        outs = ctx.compress_batch(gs, [p] * len(xs))
    for r, ref in zip(outs, refs):
        assert r.blob() == ref.blob()
    for y, ref in zip(ctx.decompress_batch(outs), refs):
        assert np.array_equal(y.cpu().numpy().view(np.uint32), ref.recon.view(np.uint32))
    for r in outs:
        r.free()
