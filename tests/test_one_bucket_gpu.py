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


@pytest.mark.parametrize("side", ["worker", "server"])
@pytest.mark.parametrize("tiles", [4, 1024])
def test_round_and_split_calls_add_the_norm_in_one_order(tiles, side):
    """The round gives what the four calls give, to the last bit of a scale: here
    the binary64 sum of the tiles' partial norms lies on the boundary between
    two binary32 scales, and adding tiles 0 to 3 one after the other gives the
    lower one, in pairs the upper."""
    import paper_2205_14473_amd as E
    from paper_2205_14473_amd.state import allocate, init_state
    d = 512 * tiles
    big = torch.zeros(d)
    big[0], big[1] = 2.0 ** 24, 1.0                     # a tie between two binary32 sums
    big[[512, 1024, 1536]] = 1.5 * 2.0 ** -30           # three eighths of a binary64 last place each
    none = E.Quant(kind=E.EA_Q_NONE, error_feedback=1)
    sign = E.Quant(kind=E.EA_Q_SCALED_SIGN, bucket=0, error_feedback=1)
    cfg = E.Config(d=d, N=1, placement=E.EA_ADAM_AT_WORKER, beta1=0.9, beta2=0.999, lr=1e-3, eps=0.0, seed=1,
                   qw=sign if side == "worker" else none, qs=sign if side == "server" else none)
    got = []
    for split in (False, True):
        rb = allocate(cfg, with_u=True)
        init_state(cfg, rb)
        rb.g.zero_()
        (rb.e_w[0] if side == "worker" else rb.e_s).copy_(big)
        if split:
            some = side == "worker"
            E.ea_worker_compress(cfg, 0, 1, rb.g[0], rb.e_w[0], rb.m_w[0], rb.v_w[0], rb.wcodes[0],
                                 rb.wscales[0] if some else None, rb.workspace)
            E.ea_server_aggregate_adam(cfg, 1, rb.wcodes, rb.wscales if some else None, rb.m, rb.v, rb.u)
            E.ea_server_compress(cfg, 1, rb.u, rb.e_s, rb.scodes, None if some else rb.sscales, rb.workspace)
            E.ea_worker_apply(cfg, rb.scodes, None if some else rb.sscales, rb.x)
        else:
            E.ea_step(cfg, 1, **rb.step_args())
        torch.cuda.synchronize()
        scale = rb.wscales if side == "worker" else rb.sscales
        got.append([t.cpu().numpy().copy() for t in (scale, rb.e_w, rb.e_s, rb.x)])
    for name, a, b in zip(("scale", "e_w", "e_s", "x"), *got):
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32)), (name, a.ravel()[:3], b.ravel()[:3])


@pytest.mark.parametrize("mode", ["step", "split"])
@pytest.mark.parametrize("what", ["zero", "subnormal", "infinite"])
@pytest.mark.parametrize("qw,qs", [(SIGN, SIGN), (STOCH(4, O.SCALE_L2), STOCH(2, O.SCALE_MAX)), (DET(3), DET(2)),
                                   (DET(6), STOCH(8, O.SCALE_L2)),
                                   (STOCH(2, O.SCALE_MAX), qfields(O.Q_SCALED_SIGN, 1, O.SCALE_L1, bucket=1024))])
def test_one_bucket_scale_zero_subnormal_or_infinite(qw, qs, what, mode):
    """Given scales that send the whole vector as zeros or need the 2^64
    pre-scale, on the specialized kernels, the generic one (server buckets of
    1024) and below and above 512 tiles.  Infinite: magnitudes whose squares
    overflow, then an infinite gradient as well, which every norm follows."""
    rng = np.random.default_rng(3)
    N = 3
    for d in (512 * 3 + 65, 513 * 512 + 1):
        pair = Pair(d, N, qw, qs, O.ADAM_AT_SERVER, seed=6, eps=0.0)
        sgn = rng.choice(np.array([-1.0, 1.0], np.float32), size=(N, d))
        g = np.zeros((N, d), np.float32)
        if what == "subnormal":
            g = sgn * (rng.integers(0, 215, (N, d)) * 2.0 ** -149).astype(np.float32)
        elif what == "infinite":
            g = sgn * rng.uniform(2.0, 3.0, (N, d)).astype(np.float32) * np.float32(1e38)
        for t in range(1, 3):
            if what == "infinite" and t == 2:
                g[:, 7] = np.inf
            pair.step(t, g)
            got = pair.rb.wscales.cpu().numpy()[:, 0]
            if what != "infinite":
                assert (got < 2.0 ** -126).all()
                assert what == "subnormal" or (got == 0).all()
        if what == "infinite":
            assert np.isinf(got).all()
        pair.check_tie_budget()
