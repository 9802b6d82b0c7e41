"""The eight-lane Huffman decode against the CPU oracle where its workgroups cross field boundaries: more units of
work than the chip holds workgroups, so each takes chunks of several fields, with their own code books, chunk sizes
and lengths."""
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


def fields(count, seed):
    """Fields of one, a few and a few hundred chunks, most chunks' last parts short, each with a spread of its own."""
    rng = np.random.default_rng(seed)
    out = []
    for i in range(count):
        n = int(rng.choice([1, 63, 64, 65, 255, 257, 3000, 8191, 40000]))
        out.append((np.cumsum(rng.normal(size=n)) * 10.0 ** rng.integers(-2, 3)).astype(np.float32))
    return out


@pytest.mark.parametrize("chunks", [(256,), (512,), (1024,), (2048,), (256, 512, 1024, 2048)])
def test_workgroups_cross_fields(ctx, chunks):
    # at least eight units a field: 360 fields are more than the 2048 workgroups that eight a CU would hold
    import torch
    xs = fields(360, sum(chunks))
    params = [dict(chunk=chunks[i % len(chunks)], eb=[1e-2, 1e-3, 1e-4][i % 3]) for i in range(len(xs))]
    refs = [O.compress(x, O.Params(shape=x.shape, **p)) for x, p in zip(xs, params)]
    print("\n[decode] %d fields, chunks %s" % (len(xs), chunks), flush=True)
    outs = ctx.compress_batch([torch.from_numpy(x).cuda() for x in xs], params)
    for ys in (ctx.decompress_batch(outs), ctx.decompress_batch(outs[::-1])[::-1]):
        for y, ref in zip(ys, refs):
            assert np.array_equal(y.cpu().numpy().view(np.uint32), ref.recon.view(np.uint32))
    for r in outs:
        r.free()


@pytest.mark.parametrize("chunk", [256, 2048])
def test_units_of_chunks(ctx, chunk):
    # a chunk's place is counted from its unit of 32, whose first word lies in the first two chunks' records: fields
    # that end at each place of a unit, the largest words a unit has (random codes of a wide range), alone and together
    import torch
    counts = [1, 2, 3, 31, 32, 33, 34, 63, 64, 65, 66, 97, 129, 161]
    xs = [np.random.default_rng(n).integers(-1000, 1000, chunk * n - n % 3).astype(np.float32) for n in counts]
    kw = dict(chunk=chunk, eb=0.5, eb_mode=0, R=1024)
    refs = [O.compress(x, O.Params(shape=x.shape, **kw)) for x in xs]
    gk = dict(chunk=chunk, eb=0.5, eb_mode=0, radius=1024)
    print("\n[decode] units, chunk %d" % chunk, flush=True)
    gs = [torch.from_numpy(x).cuda() for x in xs]
    rs = ctx.compress_batch(gs, [gk] * len(xs))
    ones = [ctx.compress(g, **gk) for g in gs]
    for ys in (ctx.decompress_batch(rs), [ctx.decompress(r) for r in ones]):
        for y, ref in zip(ys, refs):
            assert np.array_equal(y.cpu().numpy().view(np.uint32), ref.recon.view(np.uint32))
    for r in rs + ones:
        r.free()


@pytest.mark.parametrize("chunks", [32 * 255, 32 * 768 - 1, 32 * 768 + 1, 32 * 1537])
def test_one_field_in_turn(ctx, chunks):
    # one field's units taken in turn by a grid of fewer, as many and more workgroups than units
    import torch
    x = np.random.default_rng(chunks).normal(size=chunks * 256 - 100).astype(np.float32)
    x[::7] = 0.0
    kw = dict(chunk=256, eb=1e-3)
    ref = O.compress(x, O.Params(shape=x.shape, **kw))
    print("\n[decode] one field, %d chunks" % chunks, flush=True)
    r = ctx.compress(torch.from_numpy(x).cuda(), **kw)
    assert np.array_equal(ctx.decompress(r).cpu().numpy().view(np.uint32), ref.recon.view(np.uint32))
    r.free()


def uploads(ctx, xs, params):
    refs = [O.compress(x, O.Params(shape=x.shape, **p)) for x, p in zip(xs, params)]
    return refs, [ctx.upload(r.blob()) for r in refs]


@pytest.mark.parametrize("count", [1, 9, 64, 65, 90])
@pytest.mark.parametrize("radius", [2, 100, 512, 1024])
def test_uploaded(ctx, count, radius):
    # without the encoder's offsets: one lane a chunk, runs of symbols up to 64 blocks (256 CUs) of short codes,
    # single ones otherwise; short and long fields, from almost all one symbol to almost none alike
    rng = np.random.default_rng(count + radius)
    xs, params = [], []
    for i in range(count):
        n = int(rng.choice([1, 2, 3, 4, 5, 31, 33, 255, 256, 257, 1023, 3000, 8191, 60000]))
        rough = np.cumsum(rng.normal(size=n))
        x = [rough, np.where(rng.random(n) < 0.02, rough, 0.0), np.zeros(n), rng.normal(size=n)][i % 4]
        xs.append(x.astype(np.float32))
        params.append(dict(chunk=[256, 512, 1024, 2048][i // 4 % 4], eb=[1e-2, 1e-3, 1e-4][i % 3], R=radius))
    refs, ups = uploads(ctx, xs, params)
    print("\n[decode] %d uploads, radius %d" % (count, radius), flush=True)
    for y, r, ref in zip(ctx.decompress_batch(ups), ups, refs):
        assert np.array_equal(y.cpu().numpy().view(np.uint32), ref.recon.view(np.uint32))
        if count <= 9:   # alone, by its own codes' lengths
            z = ctx.decompress(r).cpu().numpy()
            assert np.array_equal(z.view(np.uint32), ref.recon.view(np.uint32))
        r.free()


def test_uploaded_with_long_codes(ctx):
    # Fibonacci counts: codes of every length, the longest past the look-up table
    x = synth.fib_spikes((96, 96, 96), n=20)
    refs, ups = uploads(ctx, [x], [dict(eb=0.5, eb_mode=0)])
    assert refs[0].code_len.max() > 13
    print("\n[decode] long codes", flush=True)
    y = ctx.decompress(ups[0]).cpu().numpy()
    assert np.array_equal(y.view(np.uint32), refs[0].recon.view(np.uint32))
    ups[0].free()


@pytest.mark.parametrize("every", [40, 400, 40000])
@pytest.mark.parametrize("shape", [(200000,), (400, 500), (40, 70, 71)])
def test_outliers_scattered(ctx, every, shape):
    # more and fewer outliers than one in 64 points: scattered by the prologue or by the decode, alone and in a batch
    import torch
    rng = np.random.default_rng(every)
    x = np.zeros(shape, np.float32)
    at = rng.choice(x.size, x.size // every, replace=False)
    x.ravel()[at] = rng.normal(size=at.size) * 100
    kw = dict(eb=1e-3, eb_mode=0, chunk=256)
    ref = O.compress(x, O.Params(shape=x.shape, **kw))
    assert (64 * len(ref.outlier_idx) > x.size) == (every == 40)
    print("\n[decode] %s, %d outliers" % (shape, len(ref.outlier_idx)), flush=True)
    r = ctx.compress(torch.from_numpy(x).cuda(), **kw)
    for y in [ctx.decompress(r)] + list(ctx.decompress_batch([r] * 3)):
        assert np.array_equal(y.cpu().numpy().view(np.uint32), ref.recon.view(np.uint32))
    r.free()


@pytest.mark.parametrize("at", [0, 3, 7])
def test_outliers_of_one_field(ctx, at):
    # a batch in which one field is nothing but outliers and the others have none: each unit scatters its own field's
    import torch
    xs = [np.zeros((20, 30, 40 + i), np.float32) for i in range(8)]
    xs[at] = np.random.default_rng(at).normal(size=(40, 50, 61)).astype(np.float32)
    kw = dict(eb=1e-30, eb_mode=0, chunk=256)
    refs = [O.compress(x, O.Params(shape=x.shape, **kw)) for x in xs]
    assert [len(r.outlier_idx) > 0 for r in refs] == [i == at for i in range(8)]
    print("\n[decode] outliers of field %d" % at, flush=True)
    rs = ctx.compress_batch([torch.from_numpy(x).cuda() for x in xs], [kw] * 8)
    outs = [torch.full(x.shape, float("nan"), device="cuda") for x in xs]
    for y, ref in zip(ctx.decompress_batch(rs, outs), refs):
        assert np.array_equal(y.cpu().numpy().view(np.uint32), ref.recon.view(np.uint32))
    for r in rs:
        r.free()
