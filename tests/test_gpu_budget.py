"""Device byte budgets: the least budgets under which these calls ran when a result's record held the bit offsets of
its chunks' parts alone (bisected to 512 bytes), and half of each, which is refused."""
import numpy as np
import pytest

import paper_2312_05492_amd as szi
from paper_2312_05492_amd import synth

pytestmark = pytest.mark.gpu


# one compression, four results held, a batch of four compressed and restored
@pytest.mark.parametrize("shape, kw, one, held, batch", [
    ((64, 64, 64), {}, 1062912, 3598848, 5215232),
    ((64, 64, 64), dict(chunk=256), 1090048, 3698176, 5282816),
    ((128, 128, 256), {}, 14947328, 50355200, 80114688),
    ((128, 128, 256), dict(chunk=256), 15377408, 51398144, 81197056),
    ((33, 40, 50), dict(chunk=2048), 340480, 1346560, 1523712),
    ((900, 1100), {}, 3578880, 12109824, 18988032),
    ((900, 1100), dict(chunk=512, eb=1e-5), 8043520, 30164992, 37084160),
    ((33793,), {}, 211456, 832000, 835072),
    ((300001,), dict(chunk=256), 1093632, 3796480, 5753856),
    ((4000000,), {}, 11790336, 41811456, 71549952),
])
def test_calls_fit(shape, kw, one, held, batch):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    x = torch.from_numpy(np.ascontiguousarray(synth.spectral_field(shape, seed=5))).cuda()

    def compress(c):
        c.compress(x, **kw).free()

    def hold(c):
        for r in [c.compress(x, **kw) for _ in range(4)]:
            r.free()

    def both(c):
        rs = c.compress_batch([x] * 4, [kw] * 4)
        c.decompress_batch(rs)
        for r in rs:
            r.free()

    for f, budget in ((compress, one), (hold, held), (both, batch)):
        print("\n[budget] %s %s: %s under %d bytes" % (shape, kw, f.__name__, budget), flush=True)
        c = szi.Context(0, budget)
        f(c)
        assert c.bytes_in_use() <= budget
        c.close()
        c = szi.Context(0, budget // 2)
        with pytest.raises(szi.SzError) as e:
            f(c)
        assert e.value.code == -3
        c.close()
