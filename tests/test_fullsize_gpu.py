"""Full-size parity: each workload at its real d and N through ea_step (the
launch the benchmark times), in both Adam placements and for the workload's
step count, checked against the oracle on sampled bucket-aligned segments
after every step.  Every step is bucket-local, so the oracle run on a segment
(with its global element offset for the draws) is exactly the slice of a full
run (pinned on the CPU by test_segment_equals_slice_of_full_run).  Also: the
split calls give the fused call's bits, and replaying steps from saved state
is bit-identical (resume)."""
import numpy as np
import pytest

import oracle as O
import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2205_14473_amd as E  # noqa: E402
from paper_2205_14473_amd.state import allocate, init_state  # noqa: E402
from parity_util import SPARSE_KINDS, RoundCheck, Stats, configs  # noqa: E402


def _segments(d, tile, count, seed):
    ntiles = -(-d // tile)
    rng = np.random.default_rng(seed)
    picks = set(rng.choice(ntiles, size=min(count, ntiles), replace=False).tolist()) | {0, ntiles - 1}
    return [(k * tile, min(tile, d - k * tile)) for k in sorted(picks)]


class Sample:
    """Bucket-aligned segments of the d-vector and device index tensors that
    gather them (and their message words and scales) in one copy each."""

    def __init__(self, oc, d, segs):
        self.segs = segs
        bw, bs = O.code_bits(oc.qw), O.code_bits(oc.qs)
        Bw, Bs = O.bucket_len(oc.qw, d), O.bucket_len(oc.qs, d)
        # one scale per bucket, or keep values per bucket for a sparsifier
        per_w = oc.qw.keep if oc.qw.kind in SPARSE_KINDS else 1
        per_s = oc.qs.keep if oc.qs.kind in SPARSE_KINDS else 1
        sw = O.num_scales(oc.qw, d, d) > 0
        ss = O.num_scales(oc.qs, d, d) > 0
        el, ww, sc_w, wsd, sc_s = [], [], [], [], []
        self.at = []
        for n0, ln in segs:
            e0, w0, s0, v0, t0 = (sum(len(a) for a in x) for x in (el, ww, sc_w, wsd, sc_s))
            el.append(np.arange(n0, n0 + ln))
            ww.append(np.arange(n0 // 256 * 4 * bw, n0 // 256 * 4 * bw + O.msg_words(oc.qw, ln)))
            wsd.append(np.arange(n0 // 256 * 4 * bs, n0 // 256 * 4 * bs + O.msg_words(oc.qs, ln)))
            nws, nss = O.num_scales(oc.qw, d, ln), O.num_scales(oc.qs, d, ln)
            sc_w.append(np.arange(n0 // Bw * per_w, n0 // Bw * per_w + nws) if sw else np.zeros(0, np.int64))
            sc_s.append(np.arange(n0 // Bs * per_s, n0 // Bs * per_s + nss) if ss else np.zeros(0, np.int64))
            self.at.append(dict(e=slice(e0, e0 + ln), w=slice(w0, w0 + len(ww[-1])), s=slice(v0, v0 + len(wsd[-1])),
                                sw=slice(s0, s0 + len(sc_w[-1])), ss=slice(t0, t0 + len(sc_s[-1]))))
        dev = lambda a: torch.from_numpy(np.concatenate(a).astype(np.int64)).cuda()  # noqa: E731
        self.el, self.ww, self.wsd, self.sc_w, self.sc_s = dev(el), dev(ww), dev(wsd), dev(sc_w), dev(sc_s)

    def rows(self, t):
        return None if t is None else t[:, self.el].cpu().numpy()

    def vec(self, t):
        return None if t is None else t[self.el].cpu().numpy()

    def messages(self, rb):
        i64 = torch.int64
        return (rb.wcodes.view(i64)[:, self.ww].cpu().numpy().view(np.uint64),
                rb.wscales[:, self.sc_w].cpu().numpy(),
                rb.scodes.view(i64)[self.wsd].cpu().numpy().view(np.uint64),
                rb.sscales[self.sc_s].cpu().numpy())

    def put_back(self, rb, k, st):
        """Reset the GPU state of segment k to the oracle's."""
        idx = self.el[self.at[k]["e"]]
        for name in ("e_w", "m_w", "v_w"):
            if getattr(st, name) is not None:
                getattr(rb, name)[:, idx] = torch.from_numpy(getattr(st, name)).cuda()
        for name in ("e_s", "x", "m", "v"):
            if getattr(st, name) is not None:
                getattr(rb, name)[idx] = torch.from_numpy(getattr(st, name)).cuda()


S, Wk = O.ADAM_AT_SERVER, O.ADAM_AT_WORKER
FULL_CASES = [("bert", S, 100), ("bert", Wk, 100), ("resnet18", S, 50), ("resnet18", Wk, 50),
              ("resnet50", S, 50), ("resnet50", Wk, 50), ("gpt2m", S, 10), ("gpt2m", Wk, 10),
              ("bert_topk", S, 20), ("bert_topk", Wk, 20), ("bert_randk", S, 20), ("bert_topk2048", S, 20),
              ("bert_randk2048", S, 20)]


@pytest.mark.parametrize("key,placement,T", FULL_CASES,
                         ids=[f"{k}-{'server' if p == S else 'worker'}-{T}" for k, p, T in FULL_CASES])
def test_full_size_sampled(key, placement, T):
    """Each workload at its real d and N through ea_step, both placements,
    for its step count (100 for the BERT-sized round): after every step the
    sampled segments' messages and state equal the oracle's bit for bit."""
    _sampled_rounds(W.WORKLOADS[key], placement, T)


@pytest.mark.parametrize("placement", [S, Wk], ids=["server", "worker"])
@pytest.mark.parametrize("tail", [76, 77], ids=["aligned", "unaligned"])
def test_launch_in_pieces(placement, tail):
    """Launches of more than 2^20 blocks are issued in pieces.  Scaled sign on
    256-element buckets with one worker, two tiles per block: d = 2^29 + 512 + 76
    (rows 16-byte aligned) and d = 2^29 + 512 + 77 (unaligned rows) take 2^20 + 2
    blocks, the last with one ragged tile: two pieces.  The segments on both sides of the piece boundary at
    element 2^29 and of its half, the first and the last are checked against
    the oracle after every step."""
    sign = W.SIGN1(256)
    d = (1 << 29) + 2 * 256 + tail
    w = W.Workload("pieces", f"d=2^29+{512 + tail} N=1, sign 256", d, 1, sign, sign, 2, 31, "student_t")
    tile = 512
    ntiles = -(-d // tile)
    b = (1 << 29) // tile        # the first segment of the second piece
    picks = sorted({0, 1, b // 2 - 1, b // 2, b - 2, b - 1, b, b + 1, ntiles - 1})
    _sampled_rounds(w, placement, 2, [(k * tile, min(tile, d - k * tile)) for k in picks])


def _sampled_rounds(w, placement, T, segs=None):
    d, N = w.d, w.N
    key = w.key
    print(f"\n[fullsize] {w.name} placement={placement} T={T}", flush=True)
    oc, ec = configs(d, N, w.qw.fields(), w.qs.fields(), placement, w.seed, w.beta1, w.beta2, w.lr, w.eps)
    rb = allocate(ec)
    init_state(ec, rb)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(w.seed)
    torch.randn(d, generator=gen, device="cuda", out=rb.x)
    rb.x.mul_(0.02)
    tile = max(O.bucket_len(oc.qw, d), O.bucket_len(oc.qs, d), 512)
    smp = Sample(oc, d, segs if segs is not None else _segments(d, tile, 24, w.seed))
    x_host = smp.vec(rb.x)
    states = [O.State.init(oc, ln, x_host[a["e"]]) for (n0, ln), a in zip(smp.segs, smp.at)]
    stats = Stats()
    for t in range(1, T + 1):
        W.device_gradients(w, t, rb.g)
        g_host = smp.rows(rb.g)
        E.ea_step(ec, t, **rb.step_args())
        torch.cuda.synchronize()
        wc, ws, sc, ss = smp.messages(rb)
        gpu = {k: smp.rows(getattr(rb, k)) for k in ("e_w", "m_w", "v_w")}
        gpu.update({k: smp.vec(getattr(rb, k)) for k in ("e_s", "x", "m", "v")})
        tied_round = False
        for k, ((n0, ln), a) in enumerate(zip(smp.segs, smp.at)):
            st = states[k]
            out = O.step(oc, t, np.ascontiguousarray(g_host[:, a["e"]]), st, n0=n0, want_inputs=True)
            chk = RoundCheck(oc, d, n0, t, out, stats, what=f"step {t} segment {n0}: ")
            chk.messages(wc[:, a["w"]], ws[:, a["sw"]], sc[a["s"]], ss[a["ss"]])
            seg = {name: (None if v is None else (v[:, a["e"]] if v.ndim == 2 else v[a["e"]]))
                   for name, v in gpu.items()}
            chk.state(seg, st)
            if chk.tied:
                tied_round = True
                smp.put_back(rb, k, st)
                stats.resyncs += 1
        stats.tie_rounds += tied_round
        stats.steps += 1
    print(f"[fullsize] {key}: {len(smp.segs)} segments x {T} steps: {stats}", flush=True)
    assert stats.tie_rounds == 0, f"{stats.scale_ties} validated one-ulp scale ties"
    assert stats.code_ties == 0 and stats.resyncs == 0
    del rb
    torch.cuda.empty_cache()


@pytest.mark.parametrize("key,placement", [("bert", None), ("gpt2m", None), ("resnet50", None), ("bert_topk", None),
                                           ("bert", O.ADAM_AT_WORKER), ("resnet18", None),
                                           ("resnet18", O.ADAM_AT_WORKER)])
def test_full_size_split_calls_equal_fused(key, placement):
    """The four split calls at full size give, output for output, the same
    bits as ea_step: both sum the workers in ascending order and run the same
    element steps, so any difference is a decoding or indexing fault at a
    size the reduced-size parity cases do not reach."""
    w = W.WORKLOADS[key]
    pl = w.placement if placement is None else placement
    print(f"\n[fullsize split] {w.name} placement={pl}", flush=True)
    _, ec = configs(w.d, w.N, w.qw.fields(), w.qs.fields(), pl, w.seed, w.beta1, w.beta2, w.lr, w.eps)
    a, b = allocate(ec), allocate(ec, with_u=True)
    init_state(ec, a)
    init_state(ec, b)
    nsw, nss = E.ea_msg_scales(ec.qw, w.d) > 0, E.ea_msg_scales(ec.qs, w.d) > 0
    for t in range(1, 3):
        W.device_gradients(w, t, a.g)
        E.ea_step(ec, t, **a.step_args())
        b.g.copy_(a.g)
        for i in range(w.N):
            E.ea_worker_compress(ec, i, t, b.g[i], b.e_w[i], None if b.m_w is None else b.m_w[i],
                                 None if b.v_w is None else b.v_w[i], b.wcodes[i],
                                 b.wscales[i] if nsw else None, b.workspace)
        E.ea_server_aggregate_adam(ec, t, b.wcodes, b.wscales if nsw else None, b.m, b.v, b.u)
        E.ea_server_compress(ec, t, b.u, b.e_s, b.scodes, b.sscales if nss else None, b.workspace)
        E.ea_worker_apply(ec, b.scodes, b.sscales if nss else None, b.x)
        torch.cuda.synchronize()
        for k in ("wcodes", "wscales", "scodes", "sscales", "e_w", "e_s", "m", "v", "m_w", "v_w", "x"):
            x, y = getattr(a, k), getattr(b, k)
            if x is None:
                continue
            assert torch.equal(x.view(torch.uint8), y.view(torch.uint8)), f"{key} step {t}: {k} differs"
    print(f"[fullsize split] {key}: bit-identical over 2 steps", flush=True)
    del a, b
    torch.cuda.empty_cache()


def test_resume_is_bit_identical():
    """10 steps, save, 10 more == 20 straight (draws depend on (seed, t, n) only)."""
    w = W.WORKLOADS["bert"]
    d, N = 512 * 64 + 100, 4
    _, ec = configs(d, N, w.qw.fields(), w.qs.fields(), O.ADAM_AT_SERVER, 4)
    grads = [torch.from_numpy(W.host_gradients(W.Workload("r", "r", d, N, None, None, 1, 4, "student_t"), t, d=d))
             for t in range(1, 21)]

    def run(rb, t0, t1):
        for t in range(t0, t1):
            rb.g.copy_(grads[t - 1])
            E.ea_step(ec, t, **rb.step_args())
        torch.cuda.synchronize()

    a = allocate(ec)
    init_state(ec, a)
    run(a, 1, 21)
    b = allocate(ec)
    init_state(ec, b)
    run(b, 1, 11)
    saved = {k: getattr(b, k).cpu().clone() for k in ("e_w", "e_s", "x", "m", "v")}
    c = allocate(ec)
    for k, val in saved.items():
        getattr(c, k).copy_(val)
    run(c, 11, 21)
    for k in ("e_w", "e_s", "x", "m", "v", "wcodes", "wscales", "scodes", "sscales"):
        assert np.array_equal(getattr(a, k).cpu().numpy(), getattr(c, k).cpu().numpy()), k
