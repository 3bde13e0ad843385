"""One code path takes every layout: ragged last tiles, an odd number of tiles
for two-tile blocks, tiles wholly past the end, rows of odd length and arrays
that start at any 4-byte address, on the specialized kernels of every tile
size and kind.  Each array lies between NaNs, which must not be read into a
result nor overwritten; results equal the oracle's bit for bit, as in the
other parity tests."""
import numpy as np
import pytest

import oracle as O

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU-only host
    pytest.skip("needs a GPU", allow_module_level=True)

from parity_util import Pair, qfields  # noqa: E402

SIGN = lambda b: qfields(O.Q_SCALED_SIGN, 1, O.SCALE_L1, bucket=b)  # noqa: E731
STOCH = lambda k, s, b: qfields(O.Q_STOCH_UNIFORM, k, s, bucket=b)  # noqa: E731
DET = lambda k, b: qfields(O.Q_DET_UNIFORM, k, bucket=b)  # noqa: E731
SPARSE = lambda kind, keep, b: qfields(kind, bucket=b, keep=keep)  # noqa: E731
POW2 = qfields(O.Q_POW2, kmin=-17, kmax=-11)
POW2W = qfields(O.Q_POW2, kmin=-20, kmax=-6)      # 5-bit codes
NONE = qfields(O.Q_NONE)
PAD = 64


def _shifted(t, shift, boxes):
    """t's values at `shift` floats past a 256-byte boundary, between NaNs."""
    if t is None:
        return None
    n = t.numel()
    big = torch.full((PAD + shift + n + PAD,), float("nan"), device="cuda")
    view = big[PAD + shift:PAD + shift + n].view(t.shape)
    view.copy_(t)
    boxes.append((big, PAD + shift, n))
    return view


# (tile length, worker and server quantizers): the fully specialized kernels,
# the ones specialized for both sides of wide tiles, the worker-specialized
# ones and the generic one
CASES = [
    (512, STOCH(4, O.SCALE_L2, 512), STOCH(4, O.SCALE_L2, 512)), (512, STOCH(2, O.SCALE_MAX, 512), STOCH(2, O.SCALE_MAX, 512)),
    (512, SPARSE(O.Q_TOPK, 16, 512), SPARSE(O.Q_TOPK, 16, 512)), (512, SPARSE(O.Q_RANDK, 16, 512), SPARSE(O.Q_RANDK, 16, 512)),
    (2048, SIGN(2048), SIGN(2048)), (1024, STOCH(2, O.SCALE_MAX, 1024), SIGN(1024)),
    (2048, SPARSE(O.Q_TOPK, 64, 2048), SPARSE(O.Q_TOPK, 64, 2048)),
    (2048, SPARSE(O.Q_RANDK, 64, 2048), SPARSE(O.Q_RANDK, 64, 2048)), (1024, SPARSE(O.Q_RANDK, 40, 1024), SPARSE(O.Q_RANDK, 40, 1024)),
    (1024, STOCH(8, O.SCALE_MAX, 1024), STOCH(8, O.SCALE_MAX, 1024)), (256, SIGN(256), SIGN(256)),
    (256, STOCH(4, O.SCALE_L2, 256), DET(3, 256)), (512, DET(3, 512), POW2), (512, POW2, NONE), (512, NONE, POW2),
    (256, DET(8, 256), POW2W), (512, DET(4, 512), DET(7, 512)), (1024, DET(6, 1024), POW2W), (2048, POW2W, DET(5, 2048)),
    (512, DET(5, 0), DET(8, 0)), (1024, DET(5, 256), STOCH(4, O.SCALE_L2, 1024)), (512, SIGN(0), DET(2, 0)), (2048, POW2, STOCH(1, O.SCALE_L2, 2048)),
]


@pytest.mark.parametrize("mode", ["step", "split"])
@pytest.mark.parametrize("tile,qw,qs", CASES)
def test_any_layout(tile, qw, qs, mode):
    rng = np.random.default_rng(5)
    sizes = [tile + 1, 2 * tile - 3, 3 * tile, 2 * tile + tile // 2 + 2]
    for j, d in enumerate(sizes):
        N = (3, 9, 1, 18)[j]
        placement = (O.ADAM_AT_SERVER, O.ADAM_AT_WORKER)[j % 2]
        pair = Pair(d, N, qw, qs, placement, seed=3 + j, mode=mode)
        boxes = []
        for k, name in enumerate(("g", "e_w", "m_w", "v_w", "m", "v", "e_s", "x", "u")):
            setattr(pair.rb, name, _shifted(getattr(pair.rb, name), (j + k) % 4, boxes))
        for t in range(1, 4):
            pair.step(t, (1e-3 * rng.standard_t(3, (N, d))).astype(np.float32))
        pair.check_tie_budget()
        for big, off, n in boxes:
            assert bool(torch.isnan(big[:off]).all()) and bool(torch.isnan(big[off + n:]).all()), (d, "written outside")
