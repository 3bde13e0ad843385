"""One bucket over the vector: scales from partial norms, formed by each wave
while the vector has at most 512 tiles and by a launch of their own above, on
the kernels specialized for a given scale and on the generic one.  Sizes at
the edges of a tile, of a partial's block of tiles and of the 512-tile rule,
against the oracle bit for bit."""
import numpy as np
import pytest

import oracle as O

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU-only host
    pytest.skip("needs a GPU", allow_module_level=True)

from parity_util import Pair, qfields  # noqa: E402

SIGN = qfields(O.Q_SCALED_SIGN, 1, O.SCALE_L1, bucket=0)
STOCH = lambda k, s: qfields(O.Q_STOCH_UNIFORM, k, s, bucket=0)  # noqa: E731
DET = lambda k: qfields(O.Q_DET_UNIFORM, k, bucket=0)  # noqa: E731


@pytest.mark.parametrize("mode", ["step", "split", "graph"])
@pytest.mark.parametrize("d", [1, 511, 512 * 4, 512 * 4 + 1, 512 * 512, 512 * 512 + 1, 600 * 512 + 7])
@pytest.mark.parametrize("qw,qs", [(SIGN, SIGN), (STOCH(4, O.SCALE_L2), DET(2)), (DET(3), STOCH(8, O.SCALE_MAX)),
                                   (STOCH(1, O.SCALE_MAX), STOCH(2, O.SCALE_L2)), (DET(6), SIGN)])
def test_one_bucket(d, qw, qs, mode):
    rng = np.random.default_rng(d)
    N = 3 if d > 4000 else 18
    sched = dict(kind=O.SCHED_CONSTANT) if mode == "graph" else None
    pair = Pair(d, N, qw, qs, (O.ADAM_AT_SERVER, O.ADAM_AT_WORKER)[d % 2], seed=4, mode=mode, sched=sched)
    for t in range(1, 4):
        pair.step(t, (1e-2 * rng.standard_normal((N, d))).astype(np.float32))
    pair.check_tie_budget()


def test_one_bucket_worker_with_bucketed_server():
    """The worker's scale on tiles of the server's bucket size."""
    rng = np.random.default_rng(2)
    for b, d in ((256, 512 * 256 + 3), (1024, 5 * 1024 - 1), (2048, 257 * 2048 + 9)):
        pair = Pair(d, 2, SIGN, qfields(O.Q_STOCH_UNIFORM, 4, O.SCALE_L2, bucket=b), O.ADAM_AT_SERVER, seed=5)
        for t in range(1, 3):
            pair.step(t, (1e-2 * rng.standard_normal((2, d))).astype(np.float32))
        pair.check_tie_budget()
