"""GPU parity of the head's training objective (Section 3.3, Equation 3): per-row
KL(softmax(l_{t-1}) || softmax(l_t + delta_t)) and its gradient with respect to the student
logits, through the C-ABI, against the fp64 oracle.

Inputs: teacher = the seeded prior logits of denoising step 1, student = those of step 0 plus a
seeded N(0, 0.5) stand-in residual (a trained head makes the two close; a second case uses
teacher + residual so that the loss is small and cancellation in it is exercised).

Tolerances (fp32 arithmetic with the hardware exponential, |logit| < ~40, V <= 151936):
every exponential carries a relative error of a few 2^-24 plus |x - lse| 2^-24 from its rounded
argument, i.e. < 4e-6 relative; sums of V such terms in a tree keep that relative error.
  loss:  a_T/s_T, lse_T and lse_S are each ~|lse| <= 20 accurate to ~1e-5 absolute, their
         combination to < 1e-4 absolute:  |loss_gpu - loss_orc| <= 1e-4 + 1e-4 |loss_orc|.
  grad:  scale (q - p) with p, q <= 1:    |g_gpu - g_orc| <= scale (2e-5 (p + q) + 1e-12).
"""
import ctypes as C

import numpy as np
import pytest
import torch
from scipy.special import softmax

import mrp_inputs as mi
import oracle as orc
import paper_2605_18817_amd as mrp
from harness import library_rule

pytestmark = pytest.mark.gpu


def _inputs(cfg, seqs, close):
    t = mi.logits0(cfg, seqs, step=1)
    if close:
        s = t + mi.residual(cfg, seqs)
    else:
        s = mi.logits0(cfg, seqs, step=0) + mi.residual(cfg, seqs)
    return t, np.ascontiguousarray(s, dtype=np.float32)


def _check(t, s, mask, scale, loss_g, grad_g, rows=None):
    rows = np.arange(t.shape[0]) if rows is None else rows
    m = None if mask is None else np.ascontiguousarray(mask[rows])
    loss_o, grad_o = orc.kl_loss(np.ascontiguousarray(t[rows]), np.ascontiguousarray(s[rows]), m, scale)
    np.testing.assert_allclose(loss_g[rows], loss_o, rtol=1e-4, atol=1e-4 * abs(scale))
    if grad_g is not None:
        p = softmax(t[rows].astype(np.float64), axis=1)
        q = softmax(s[rows].astype(np.float64), axis=1)
        err = np.abs(grad_g[rows] - grad_o)
        bound = abs(scale) * (2e-5 * (p + q) + 1e-12)
        assert np.all(err <= bound), float((err / bound).max())
        if m is not None:
            assert np.all(grad_g[rows][m == 0] == 0.0) and np.all(loss_g[rows][m == 0] == 0.0)
    return loss_o


@pytest.mark.parametrize("V,M,close", [(4096, 4, False), (4096, 4, True), (5003, 24, False), (8192, 16, True),
                                       (33000, 8, False), (151936, 8, True)])
def test_kl_loss_and_gradient_match_oracle(V, M, close):
    cfg = mi.config(0, V=V, B=M // 4, L=4)
    ctx = mrp.MrpContext(cfg.d, V, M, cfg.L)
    try:
        t, s = _inputs(cfg, None, close)
        mask = (np.arange(M) % 3 != 1).astype(np.uint8)
        t_d, s_d = torch.from_numpy(t).cuda(), torch.from_numpy(s).cuda()
        for mk, scale in ((None, 1.0), (mask, 0.25)):
            loss = torch.full((M,), 7.0, dtype=torch.float32, device="cuda")
            grad = torch.full((M, V), 7.0, dtype=torch.float32, device="cuda")
            mk_d = None if mk is None else torch.from_numpy(mk).cuda()
            ctx.kl_loss(M, t_d, s_d, mk_d, scale, loss, grad)
            torch.cuda.synchronize()
            lo = _check(t, s, mk, scale, loss.cpu().numpy(), grad.cpu().numpy())
            # forward only leaves grad alone and gives the same loss bits
            loss2 = torch.empty_like(loss)
            ctx.kl_loss(M, t_d, s_d, mk_d, scale, loss2, None)
            torch.cuda.synchronize()
            assert torch.equal(loss, loss2)
        print(f"\n[kl V={V} M={M} close={close}] mean loss {lo.mean():.4f}", flush=True)
    finally:
        ctx.close()


def test_kl_loss_zero_when_student_equals_teacher_up_to_a_constant():
    cfg = mi.config(0, V=10000, B=2, L=4)
    ctx = mrp.MrpContext(cfg.d, cfg.V, cfg.M, cfg.L)
    try:
        t = mi.logits0(cfg)
        t_d = torch.from_numpy(t).cuda()
        s_d = t_d + 2.0
        loss = torch.empty((cfg.M,), dtype=torch.float32, device="cuda")
        grad = torch.empty((cfg.M, cfg.V), dtype=torch.float32, device="cuda")
        ctx.kl_loss(cfg.M, t_d, s_d, None, 1.0, loss, grad)
        torch.cuda.synchronize()
        assert loss.abs().max().item() < 1e-4
        assert grad.abs().max().item() < 2e-5
        # row sums of the gradient vanish (both softmaxes sum to one)
        assert grad.double().sum(1).abs().max().item() < 1e-5
    finally:
        ctx.close()


def test_kl_loss_argument_errors():
    cfg = mi.config(0)
    ctx = mrp.MrpContext(cfg.d, cfg.V, cfg.M, cfg.L)
    try:
        t = torch.zeros((cfg.M, cfg.V), dtype=torch.float32, device="cuda")
        loss = torch.zeros((cfg.M,), dtype=torch.float32, device="cuda")
        assert ctx.kl_loss(cfg.M + 1, t, t, None, 1.0, loss, None, check=False) != 0
        assert ctx.kl_loss(cfg.M, None, t, None, 1.0, loss, None, check=False) != 0
        assert ctx.kl_loss(cfg.M, t.view(-1)[1:], t, None, 1.0, loss, None, check=False) != 0   # misaligned
        assert ctx.kl_loss(0, t, t, None, 1.0, loss, None, check=False) == 0
    finally:
        ctx.close()


@pytest.mark.timeout(600)
def test_kl_loss_full_size_sampled_rows():
    """Config 2's row count and vocabulary (the size the throughput figure is quoted on); the
    oracle checks a sample of rows, the rest by invariants that hold at any size."""
    cfg = mi.config(2)
    M, V = cfg.M, cfg.V
    ctx = mrp.MrpContext(256, V, M, cfg.L)
    try:
        t, s = _inputs(cfg, None, True)
        mask = (np.arange(M) % 5 != 2).astype(np.uint8)
        t_d, s_d = torch.from_numpy(t).cuda(), torch.from_numpy(s).cuda()
        loss = torch.empty((M,), dtype=torch.float32, device="cuda")
        grad = torch.empty((M, V), dtype=torch.float32, device="cuda")
        ctx.kl_loss(M, t_d, s_d, torch.from_numpy(mask).cuda(), 1.0 / M, loss, grad)
        torch.cuda.synchronize()
        rows = np.array([0, 1, 2, 517, 1022, 1023])
        loss_h = loss.cpu().numpy()
        _check(t, s, mask, 1.0 / M, loss_h, grad.cpu().numpy(), rows)
        on = mask == 1
        assert np.all(loss_h[on] > 0) and np.all(loss_h[~on] == 0)
        rs = grad.double().sum(1).abs().max().item()
        assert rs < 1e-5 / M * 4, rs
        assert torch.all(grad[torch.from_numpy(~on).cuda()] == 0)
    finally:
        ctx.close()


@pytest.mark.parametrize("V,M", [(151936, 391), (50257, 403), (50257, 259)])   # one pass, rows dealt unevenly over the counters; two passes
def test_kl_loss_over_groups_of_rows(V, M):
    g = torch.Generator(device="cuda")
    g.manual_seed(V + M)
    t = torch.empty(M, V, device="cuda").normal_(0, 2, generator=g)
    s = t + torch.empty(M, V, device="cuda").normal_(0, 0.5, generator=g)
    mask = (torch.arange(M, device="cuda") % 5 != 2).to(torch.uint8)
    loss, loss1 = torch.full((M,), 9.0, device="cuda"), torch.full((M,), 9.0, device="cuda")
    grad = torch.full((M + 1, V), 9.0, device="cuda")
    ctx = mrp.MrpContext(128, V, M, 1)
    ctx.kl_loss(M, t, s, mask, 0.5, loss, grad[:M])
    ctx.kl_loss(M, t, s, mask, 0.5, loss1)
    on = mask.double().unsqueeze(1)
    p, q = torch.log_softmax(t.double(), 1), torch.log_softmax(s.double(), 1)
    want = 0.5 * ((p.exp() * (p - q)).sum(1) * on[:, 0])
    for got in (loss, loss1):
        assert bool(((got - want).abs() <= 0.5 * 1e-4 + 1e-4 * want).all())
    bound = 0.5 * (2e-5 * (p.exp() + q.exp()) + 1e-12) * on       # as above; rows that are off: exactly zero
    assert bool(((grad[:M] - 0.5 * (q.exp() - p.exp()) * on).abs() <= bound).all())
    assert bool((grad[M] == 9.0).all())
    ctx.close()


@pytest.mark.parametrize("V,M", [(4096, 2048), (4096, 2049), (8193, 1024), (8193, 1023), (151936, 108), (151936, 107), (65537, 230),
                                 (262147, 63)])     # both sides of 2048 tiles; 1, 2, 9, 19 and 33 tiles a row: 7 to 3 counters
def test_gradient_in_one_pass_and_two(V, M):
    """The one-pass form and the two-pass form give the bits of the forward pass for the loss, for any order of rows on and off,
    in place, and again on the same context (its words are cleared)."""
    nq = library_rule("_ZN3mrp11kl_countersEiii", C.c_int, *[C.c_int] * 3)(M, -(-V // 8192), 256)
    assert (nq > 0) == (M * -(-V // 8192) >= 2048)
    g = torch.Generator(device="cuda")
    g.manual_seed(V + M)
    t = torch.empty(M, V, device="cuda").normal_(0, 2, generator=g)
    s = t + torch.empty(M, V, device="cuda").normal_(0, 0.5, generator=g)
    p, q = torch.log_softmax(t.double(), 1), torch.log_softmax(s.double(), 1)
    ctx = mrp.MrpContext(128, V, M, 1)
    for mask in (None, (torch.rand(M, device="cuda", generator=g) < 0.5).to(torch.uint8)):
        on = torch.ones(M, 1, device="cuda", dtype=torch.double) if mask is None else mask.double().unsqueeze(1)
        loss, loss1 = torch.full((M,), 9.0, device="cuda"), torch.full((M,), 9.0, device="cuda")
        ctx.kl_loss(M, t, s, mask, 0.5, loss1)
        for grad in (torch.full((M, V), 9.0, device="cuda"), s.clone()):      # the second over the student's own logits
            src = grad if bool((grad == s).all()) else s
            ctx.kl_loss(M, t, src, mask, 0.5, loss, grad)
            assert torch.equal(loss, loss1)
            bound = 0.5 * (2e-5 * (p.exp() + q.exp()) + 1e-12) * on
            assert bool(((grad - 0.5 * (q.exp() - p.exp()) * on).abs() <= bound).all())
    ctx.close()


def _launch():
    """The loss with a number of CUs and of looks of its own (the library's: the stream's CUs)."""
    return library_rule("_ZN3mrp14launch_kl_lossEiiPKfS1_PKhfPfmS4_S4_iiP12ihipStream_t", C.c_int, C.c_int, C.c_int, *[C.c_void_p] * 3,
                        C.c_float, C.c_void_p, C.c_size_t, C.c_void_p, C.c_void_p, C.c_int, C.c_int, C.c_void_p)


def _tensors(V, M):
    g = torch.Generator(device="cuda")
    g.manual_seed(V)
    t = torch.empty(M, V, device="cuda").normal_(0, 2, generator=g)
    return t, t + torch.empty(M, V, device="cuda").normal_(0, 0.5, generator=g)


@pytest.mark.parametrize("V,M", [(151936, 108), (8193, 1024)])
def test_one_pass_without_waiting(V, M):
    """A workgroup that finds its row's other partials missing takes them itself: with no patience at all, the same bits, also
    over the student's own logits."""
    launch = _launch()
    t, s = _tensors(V, M)
    n = M * -(-V // 8192)
    words = torch.zeros(5 * n + 16 * 7, dtype=torch.int64, device="cuda")
    loss, want, grad = [torch.full((M,), 9.0, device="cuda") for _ in range(2)] + [torch.empty_like(s)]
    ctx = mrp.MrpContext(128, V, M, 1)
    ctx.kl_loss(M, t, s, None, 0.5, want, grad)
    ctx.close()
    for out in (torch.full_like(s, 9.0), s):
        assert launch(M, V, t.data_ptr(), s.data_ptr(), None, 0.5, words.data_ptr(), n, loss.data_ptr(), out.data_ptr(), 256, 0,
                      torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
        assert torch.equal(loss, want) and torch.equal(out, grad)


@pytest.mark.parametrize("V,M", [(151936, 391), (151936, 135), (151936, 134), (1100000, 40), (4000000, 17)])
def test_two_passes_over_groups_of_rows(V, M):
    """Rows whose tiles are too many for the places that may wait (32 CUs; a vocabulary above a million on any number) take two
    passes, in groups of rows from one and a half of them on (135 rows of 151936), with the bits of the forward pass for
    the loss, also in place and with rows off."""
    nCU = 32 if V < 1000000 else 256
    assert library_rule("_ZN3mrp11kl_countersEiii", C.c_int, *[C.c_int] * 3)(M, -(-V // 8192), nCU) == 0
    launch = _launch()
    t, s = _tensors(V, M)
    n = M * -(-V // 8192)
    words = torch.zeros(5 * n + 16 * 7, dtype=torch.int64, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    mask = (torch.arange(M, device="cuda") % 5 != 2).to(torch.uint8)
    loss, want = torch.full((M,), 9.0, device="cuda"), torch.full((M,), 9.0, device="cuda")
    assert launch(M, V, t.data_ptr(), s.data_ptr(), mask.data_ptr(), 0.5, words.data_ptr(), n, want.data_ptr(), None, nCU, 9, st) == 0
    lt, ls = torch.logsumexp(t.double(), 1, keepdim=True), torch.logsumexp(s.double(), 1, keepdim=True)
    s0 = s.clone()
    for out in (torch.full((M + 1, V), 9.0, device="cuda")[:M], s):
        assert launch(M, V, t.data_ptr(), s.data_ptr(), mask.data_ptr(), 0.5, words.data_ptr(), n, loss.data_ptr(), out.data_ptr(),
                      nCU, 9, st) == 0
        torch.cuda.synchronize()
        assert torch.equal(loss, want)
        for i in range(M):
            p, q = (t[i].double() - lt[i]).exp(), (s0[i].double() - ls[i]).exp()
            bound = 0.5 * (2e-5 * (p + q) + 1e-12)                # as above; rows that are off: exactly zero
            assert bool(((out[i] - 0.5 * (q - p) * float(mask[i])).abs() <= bound * float(mask[i])).all()), i


@pytest.mark.parametrize("cus", [8, 128, 192])
def test_stream_of_few_compute_units(cus):
    """On a stream limited to some CUs the library counts those: two passes below 128."""
    V, M = 50257, 1024
    torch.zeros(1, device="cuda")
    hip = C.CDLL(next(ln.split()[-1] for ln in open("/proc/self/maps") if "libamdhip64" in ln))
    words = (C.c_uint32 * 8)(*[(1 << max(0, min(32, cus - 32 * i))) - 1 for i in range(8)])
    handle = C.c_void_p()
    assert hip.hipExtStreamCreateWithCUMask(C.byref(handle), C.c_uint32(8), words) == 0
    count = library_rule("_ZN3mrp10stream_cusEP12ihipStream_ti", C.c_int, C.c_void_p, C.c_int)
    assert count(handle, 256) == cus and count(None, 256) == 256
    t, s = _tensors(V, M)
    out = [(torch.full((M,), 9.0, device="cuda"), torch.full((M, V), 9.0, device="cuda")) for _ in range(2)]
    ctx = mrp.MrpContext(128, V, M, 1)
    ctx.kl_loss(M, t, s, None, 0.5, *out[0])
    torch.cuda.synchronize()
    stream = torch.cuda.ExternalStream(handle.value)
    with torch.cuda.stream(stream):
        ctx.kl_loss(M, t, s, None, 0.5, *out[1])
    stream.synchronize()
    lt, ls = torch.logsumexp(t.double(), 1, keepdim=True), torch.logsumexp(s.double(), 1, keepdim=True)
    p, q = (t.double() - lt).exp(), (s.double() - ls).exp()
    for loss, grad in out:
        assert torch.equal(loss, out[0][0])
        assert bool(((grad - 0.5 * (q - p)).abs() <= 0.5 * (2e-5 * (p + q) + 1e-12)).all())     # as above
    graph = torch.cuda.CUDAGraph()                                 # the stream is asked for its CUs under capture, too
    with torch.cuda.graph(graph):
        ctx.kl_loss(M, t, s, None, 0.5, *out[1])
    for _ in range(3):
        out[1][1].fill_(9.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    ctx.close()
    del stream
    assert hip.hipStreamDestroy(handle) == 0
