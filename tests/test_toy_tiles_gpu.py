"""The toy problem's matrix-core sums where their shape changes: one block and
two, the edges of 16-row groups, of 32- and 64-column blocks and of message
chunks, the last worker of a pass and the first of the next, and both column
widths at their border.  Gradients against binary64 sums in plain torch (each
rounded once: within one unit in the last place, the sums' order being free),
the round against ea_step's on the same gradients bit for bit, and message
words written whole (their buffers start filled with ones)."""
import math

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU-only host
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2205_14473_amd as E  # noqa: E402
from paper_2205_14473_amd.state import allocate, init_state  # noqa: E402


def _quant(kind):
    if kind == "none":
        return E.Quant(kind=E.EA_Q_NONE, error_feedback=1)
    lo, hi = {"ex2": (-17, -11), "wide": (-126, 127)}[kind]     # 4- and 9-bit codes
    return E.Quant(kind=E.EA_Q_POW2, pow2_kmin=lo, pow2_kmax=hi, error_feedback=1)


@pytest.mark.parametrize("d,N,kind", [
    (1, 1, "ex2"), (15, 15, "wide"), (16, 16, "ex2"), (33, 2, "ex2"), (64, 14, "wide"), (65, 15, "ex2"),
    (96, 16, "wide"), (255, 30, "ex2"), (257, 31, "none"), (500, 10, "wide"), (2048 + 31, 3, "ex2"),
    (16320, 2, "ex2"), (16321, 3, "wide"), (16415, 15, "ex2")])
def test_tile_edges(d, N, kind):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d + N)
    rnd = lambda *s: torch.randn(s, generator=gen, device="cuda")  # noqa: E731
    A, xs, xi, x = rnd(d, d), rnd(d) * math.sqrt(0.1), rnd(N, d) * math.sqrt(0.1), rnd(d)
    q = _quant(kind)
    at = E.EA_ADAM_AT_WORKER if d % 2 else E.EA_ADAM_AT_SERVER
    cfg = E.Config(d=d, N=N, placement=at, beta1=0.9, beta2=0.99, lr=1e-4, eps=1e-8, seed=1, qw=q, qs=q)
    a, b = allocate(cfg), allocate(cfg)
    for rb in (a, b):
        init_state(cfg, rb)
        rb.x.copy_(x)
        rb.wcodes.view(torch.int64).fill_(-1)
        rb.scodes.view(torch.int64).fill_(-1)
    ws = torch.empty(E.ea_toy_workspace_bytes(d), dtype=torch.uint8, device="cuda")
    gsq, g = torch.zeros(1, dtype=torch.float64, device="cuda"), torch.empty((N, d), device="cuda")
    E.ea_toy_step(cfg, 3, A, xs, xi, a.e_w, a.m_w, a.v_w, a.m, a.v, a.e_s, a.x, a.wcodes, a.scodes, gsq, g, ws)
    r = torch.stack([A[i].double() @ x.double() for i in range(d)]) if d < 64 else \
        torch.cat([c.double() @ x.double() for c in A.split(2048)])
    r = r - xs.double()
    want, full = torch.zeros(N, d, dtype=torch.float64, device="cuda"), torch.zeros(d, dtype=torch.float64,
                                                                                  device="cuda")
    for k, c in zip(range(0, d, 2048), A.split(2048)):
        c = c.double()
        want += (r[k:k + 2048] - xi[:, k:k + 2048].double()) @ c
        full += r[k:k + 2048] @ c
    # binary64 sums of d terms differ by at most about d 2^-53 of the sum of
    # magnitudes (sqrt(d) times a result): far below the half unit of the
    # one binary32 rounding except where a sum cancels
    scale = 2.0 * want.abs().amax().item()
    assert torch.all((g.double() - 2.0 * want).abs() <= 2.0 ** -24 * (2.0 * want).abs() + d * 2.0 ** -52 * scale)
    assert gsq.item() == pytest.approx((2.0 * full).square().sum().item(), rel=1e-12)
    b.g.copy_(g)
    E.ea_step(cfg, 3, **b.step_args())
    torch.cuda.synchronize()
    if kind == "none" and d % 2:                 # the last word's upper half lies past d
        a.wcodes, b.wcodes = (t.wcodes.view(torch.float32)[:, :d] for t in (a, b))
        a.scodes, b.scodes = (t.scodes.view(torch.float32)[:d] for t in (a, b))
    for name in ("wcodes", "scodes", "e_w", "e_s", "x", "m", "v", "m_w", "v_w"):
        u, v = getattr(a, name), getattr(b, name)
        if u is not None:
            dt = torch.int64 if u.dtype == torch.uint64 else torch.int32
            assert torch.equal(u.contiguous().view(dt), v.contiguous().view(dt)), name
