"""The bytes that the sampler reports for a direct product: the fields, the
masks, the class words and the records, each once."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from test_gpu_taps import DEV, domain, fc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("uniform", [True, False])
@pytest.mark.parametrize("dims,at", [((40, 24, 20), 2.5), ((70, 48), 1.5), ((300,), 2.5)])
def test_bytes_of_a_product(dims, at, uniform):
    """On a periodic box every node is interior where the volumes are uniform
    (records 0 and 1 only) and has a record of its own where no two are alike."""
    f = fc()
    h, chi, _, vol = domain(dims, at, "periodic")
    if uniform:
        vol = np.full(chi.shape, np.prod(h))
    g = f.Problem(dims, h, (at,) * len(dims), 1, chi, None, vol, device=DEV)
    r = int(np.ceil(at)) - 1
    tile = 256 if len(dims) == 1 else 32
    words = ((dims[0] + tile - 1) // tile * (tile // 2) + r) * int(np.prod(dims[1:]))
    s = len(dims) + 1
    for dtype, elem in ((torch.float32, 4), (torch.float64, 8)):
        per = 16 // elem
        pitch = (s * (s + 1) // 2 + per - 1) // per * per * elem   # M's upper triangle, whole 16 bytes
        # the reference node of the classes shares its volume with itself alone
        own = 0 if uniform else 2 * words
        for nrhs in (1, 3):
            x = torch.ones((nrhs,) + chi.shape, dtype=dtype, device=DEV)
            g.profile(True)
            g.apply("K_FULL", x)
            g.profile(False)
            kinds = g.profile_read()
            (name, (n, ms, by)), = kinds.items()
            want = nrhs * x[0].numel() * (2 * elem + 2) + 4 * words + (own + 2) * pitch
            print(f"  {dims} {name} x{nrhs}: {by:.0f} bytes, {want} expected", flush=True)
            # (the words that cover the reference node have no record for it)
            assert n == 1 and want - (0 if uniform else 8 * pitch) <= by <= want
    g.close()
