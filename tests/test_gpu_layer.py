"""The decoder-layer kernels (libcplayer.so) and the layer around the
attention step against the fp64 reference of oracle/layer.py, on the GPU.

Tolerances.  Each kernel computes in fp32 (the rotation angle is reduced in
fp64 before an fp32 sine and cosine) and
rounds its output once to bf16, so its error is at most half a bf16 ulp of
the result (2^-9 relative) plus fp32 noise: the tests allow 2^-8 relative
plus a small absolute term.  The whole layer rounds to bf16 at every kernel
and GEMM boundary (about eight roundings on the longest path, each 2^-9
relative, accumulated through fp32 GEMMs): the test bounds the error by 4 %
of the output's RMS at the maximum and 0.6 % on average."""

import math

import numpy as np
import pytest
import torch

from oracle import layer as ref
from paper_2606_09061_amd import model as M

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)


def _bf16(shape, seed, scale=1.0):
    g = torch.Generator(device="cpu").manual_seed(seed)
    return (torch.randn(*shape, generator=g) * scale).to(torch.bfloat16)


def _f64(t):
    return t.float().cpu().numpy().astype(np.float64)


def _close(got, want, rel=2.0 ** -8, abs_=1e-5):
    err = np.abs(got - want)
    bound = rel * np.abs(want) + abs_
    assert np.all(err <= bound), f"max excess {np.max(err - bound):.3e}, max err {err.max():.3e}"


@pytest.mark.parametrize("n,width", [(1, 8), (37, 4096), (5, 12288), (3, 520), (3, 1024), (5, 1032),
                                     (2, 2048), (4, 2056), (3, 4104)])
def test_rmsnorm_matches_reference(n, width):
    print(f"rmsnorm n={n} width={width}", flush=True)
    x = _bf16((n, width), 1, 3.0)
    w = _bf16((width,), 2)
    out = torch.empty_like(x, device=DEV)
    M.rmsnorm(x.to(DEV), w.to(DEV), out, 1e-6)
    torch.cuda.synchronize()
    _close(_f64(out), ref.rmsnorm(_f64(x), _f64(w), 1e-6))


def test_rmsnorm_in_place():
    _rmsnorm_in_place(1024)


@pytest.mark.parametrize("width", [2048, 4096])
def test_rmsnorm_in_place_of_held_rows(width):
    _rmsnorm_in_place(width)


def _rmsnorm_in_place(width):
    x = _bf16((9, width), 3).to(DEV)
    w = _bf16((width,), 4).to(DEV)
    want = ref.rmsnorm(_f64(x), _f64(w), 1e-6)
    M.rmsnorm(x, w, x, 1e-6)
    torch.cuda.synchronize()
    _close(_f64(x), want)


@pytest.mark.parametrize("T,hq,hkv,D", [(1, 4, 2, 128), (50, 32, 8, 128), (7, 8, 1, 64),
                                        (3, 5, 3, 128), (5, 3, 2, 64)])
def test_qkv_rope_matches_reference(T, hq, hkv, D):
    print(f"qkv_rope T={T} hq={hq} hkv={hkv} D={D}", flush=True)
    qkv = _bf16((T, (hq + 2 * hkv) * D), 5)
    qw, kw = _bf16((D,), 6), _bf16((D,), 7)
    pos = torch.from_numpy(np.random.default_rng(8).integers(0, 32768, T).astype(np.int32))
    q = torch.empty(T, hq, D, dtype=torch.bfloat16, device=DEV)
    k = torch.empty(T, hkv, D, dtype=torch.bfloat16, device=DEV)
    v = torch.empty(T, hkv, D, dtype=torch.bfloat16, device=DEV)
    M.qkv_rope(qkv.to(DEV), qw.to(DEV), kw.to(DEV), pos.to(DEV), hq, hkv, D, 1e6, 1e-6, q, k, v)
    torch.cuda.synchronize()
    rq, rk, rv = ref.qkv_rope(_f64(qkv), _f64(qw), _f64(kw), pos.numpy(), hq, hkv, D, 1e6, 1e-6)
    _close(_f64(q), rq, abs_=1e-4)
    _close(_f64(k), rk, abs_=1e-4)
    assert torch.equal(v.cpu(), qkv.view(T, hq + 2 * hkv, D)[:, hq + hkv:])  # bit copy


@pytest.mark.parametrize("T,inter", [(1, 8), (33, 12288), (4, 1000)])
def test_swiglu_matches_reference(T, inter):
    gu = _bf16((T, 2 * inter), 9, 4.0)
    out = torch.empty(T, inter, dtype=torch.bfloat16, device=DEV)
    M.swiglu(gu.to(DEV), out)
    torch.cuda.synchronize()
    _close(_f64(out), ref.swiglu(_f64(gu)), abs_=1e-6)


def test_bad_arguments_are_rejected():
    x = torch.zeros(4, 16, dtype=torch.bfloat16, device=DEV)
    with pytest.raises(Exception):
        M.rmsnorm(x[:, 1:9], x[0, :8], x[:, :8], 1e-6)   # strided view
    lib = M.load()
    p = x.data_ptr()
    assert lib.cpl_rmsnorm(p + 2, p, p, 1, 8, 1e-6, None) != 0   # misaligned: nothing launched
    assert lib.cpl_rmsnorm(p, p, p, 1, 12, 1e-6, None) != 0      # width not a multiple of 8
    assert lib.cpl_qkv_rope(1, 1, 1, 1, 1, 1, 1, 96, 1e6, 1e-6, 1, 1, 1, None) != 0
    y = torch.zeros(64, dtype=torch.int32, device=DEV).data_ptr()
    assert lib.cpl_qkv_rope(p + 2, p, p, y, 1, 1, 1, 64, 1e6, 1e-6, p, p, p, None) != 0  # misaligned
    assert lib.cpl_swiglu(1, 1, 1, 12, None) != 0


def test_project_matches_library_and_reference():
    from paper_2606_09061_amd import model as MM
    for m_rows in (1, 32, 33):          # skinny kernel, then the tiled one
        a = _bf16((m_rows, 512), 31).to(DEV)
        w = _bf16((256, 512), 32, 0.05).to(DEV)
        x = _bf16((m_rows, 256), 33).to(DEV)
        want = _f64(x) + _f64(a) @ _f64(w).T
        MM.project(a, w, x, x)
        torch.cuda.synchronize()
        err = np.abs(_f64(x) - want)
        assert err.max() <= 2e-2 * max(1.0, float(np.abs(want).max()))


@pytest.mark.parametrize("form", ["dense", "w_strided", "a_strided", "a_negated", "out_at_8_bytes",
                                  "residual_copy", "residual_overlaps_out", "autograd", "n_odd",
                                  "side_stream"])
@pytest.mark.parametrize("rows", [20, 45])
def test_project_of_every_form(rows, form):
    """project() on tensors that the tiled kernel takes and on those that stay
    with the library, against the fp64 product: one bf16 rounding of the
    result plus fp32 sums (test_gemm_matches_reference's bound); where the
    library adds a residual after rounding, one more rounding of the product."""
    from paper_2606_09061_amd import model as MM
    N, K = (160 if form == "n_odd" else 256), 1024
    a, w, r = _bf16((rows, K), 61), _bf16((N, K), 62, 0.05), _bf16((rows, N), 63)
    ad, wd, rd = a.to(DEV), w.to(DEV), None
    out = torch.empty(rows, N, dtype=torch.bfloat16, device=DEV)
    stream = None
    if rows <= 32 and form in ("w_strided", "a_strided", "a_negated", "out_at_8_bytes"):
        pytest.skip("the skinny kernel's batch sizes: dense, plain and aligned tensors only")
    if form == "w_strided":
        wd = torch.zeros(N, K + 64, dtype=torch.bfloat16, device=DEV)[:, :K].copy_(w)
    elif form == "a_strided":
        ad = torch.zeros(rows, K + 64, dtype=torch.bfloat16, device=DEV)[:, :K].copy_(a)
    elif form == "a_negated":       # the sign is in the view, not in memory
        ad = torch._neg_view(-ad)
    elif form == "out_at_8_bytes":
        out = torch.empty(rows * N + 4, dtype=torch.bfloat16, device=DEV)[4:].view(rows, N)
    elif form == "residual_copy":
        rd = r.to(DEV)
    elif form == "residual_overlaps_out":
        if rows <= 32:
            pytest.skip("the skinny kernel's batch sizes: residual apart from out, or out itself")
        def overlapping():   # the residual lies one row further on
            buf = torch.empty((rows + 1) * N, dtype=torch.bfloat16, device=DEV)
            buf[N:] = r.to(DEV).view(-1)
            return buf[:rows * N].view(rows, N), buf[N:].view(rows, N)
        out, rd = overlapping()
        assert not MM._tiled_takes(ad, wd, out, rd)
        want, copy = overlapping()   # torch's own answer, or its refusal
        try:
            torch.addmm(copy, ad, wd.t(), out=want)
        except RuntimeError:
            with pytest.raises(RuntimeError):
                MM.project(ad, wd, out, rd)
        else:
            MM.project(ad, wd, out, rd)
            assert torch.equal(out, want)
        return
    elif form == "autograd":
        wd = torch.nn.Parameter(wd)
        with pytest.raises(RuntimeError) if rows > 32 else torch.no_grad():
            MM.project(ad, wd, out)
        if rows > 32:
            return
    elif form == "side_stream":
        stream = torch.cuda.Stream(DEV)
        stream.wait_stream(torch.cuda.current_stream(DEV))
    MM.project(ad, wd, out, rd, stream.cuda_stream if stream is not None else None)
    torch.cuda.synchronize()
    prod = _f64(a) @ _f64(w).T
    want = prod + (_f64(r) if rd is not None else 0.0)
    slack = 2.0 ** -20 * (np.abs(_f64(a)) @ np.abs(_f64(w)).T) + 2.0 ** -8 * np.abs(prod)
    err = np.abs(_f64(out) - want)
    assert np.all(err <= 2.0 ** -8 * np.abs(want) + slack + 1e-6), f"max err {err.max():.3e}"


def _torch_operands(rows=45):
    """a [rows, 1024], w [256, 1024] and a result's place, of the tiled kernel's kind."""
    return (_bf16((rows, 1024), 64).to(DEV), _bf16((256, 1024), 65, 0.05).to(DEV),
            _bf16((rows, 256), 66).to(DEV))


@pytest.mark.parametrize("handle", [False, True])
def test_project_left_to_the_library_runs_on_the_given_stream(handle):
    """A strided operand is the library's; its product follows the work on the
    stream that project() is given, not on the current one."""
    from paper_2606_09061_amd import model as MM
    a, w, x = _torch_operands()
    ws = torch.zeros(256, 1088, dtype=torch.bfloat16, device=DEV)[:, :1024]
    out = torch.zeros_like(x)
    torch.mm(a, w.t(), out=x)
    torch.cuda.synchronize()
    side = torch.cuda.Stream(DEV)
    with torch.cuda.stream(side):
        torch.cuda._sleep(20_000_000)     # milliseconds
        ws.copy_(w)
    MM.project(a, ws, out, None, side.cuda_stream if handle else side)
    side.synchronize()
    assert torch.equal(out, x)


def test_project_in_forward_mode():
    """Inside a dual level the products above the skinny kernel's batch sizes
    are torch's: refused into a given tensor, with their tangent in place."""
    import torch.autograd.forward_ad as fwd
    from paper_2606_09061_amd import model as MM
    a, w, x = _torch_operands()
    tangent = torch.randn_like(a)
    with fwd.dual_level():
        dual = fwd.make_dual(a, tangent)
        with pytest.raises(NotImplementedError):
            MM.project(dual, w, torch.empty_like(x))
        y = x.clone()
        MM.project(dual, w, y, y)
        got = fwd.unpack_dual(y).tangent
        assert got is not None and torch.equal(got, torch.mm(tangent, w.t()))


@pytest.mark.parametrize("transform", ["vmap", "jvp", "grad", "functionalize"])
def test_project_in_function_transforms(transform):
    """The wrapped tensors of torch.func have no memory of their own; the
    product above the skinny kernel's batch sizes follows them as torch's."""
    from paper_2606_09061_amd import model as MM
    a, w, x = _torch_operands()

    def f(t, product):
        y = x + 0 * t[:, :256]          # wrapped like t
        product(t, y)
        return y

    def ours(t):
        return f(t, lambda u, y: MM.project(u, w, y, y))

    def torchs(t):
        return f(t, lambda u, y: y.addmm_(u, w.t()))
    run = {"vmap": lambda g: torch.func.vmap(g)(torch.stack([a, 2 * a])),
           "jvp": lambda g: torch.stack(torch.func.jvp(g, (a,), (torch.ones_like(a),))),
           "grad": lambda g: torch.func.grad(lambda t: g(t).float().sum())(a),
           "functionalize": lambda g: torch.func.functionalize(g)(a)}[transform]
    assert torch.equal(run(ours), run(torchs))


def test_project_under_modes_traces_and_the_compiler():
    """Whoever watches torch's operations sees the products above the skinny
    kernel's batch sizes; the mode of a default device watches nothing."""
    from torch.utils.flop_counter import FlopCounterMode
    from paper_2606_09061_amd import model as MM
    a, w, x = _torch_operands()
    want = torch.empty_like(x)
    torch.mm(a, w.t(), out=want)

    def ours(t):
        out = torch.empty_like(x)
        MM.project(t, w, out)
        return out
    with FlopCounterMode(display=False) as counter:
        ours(a)
    assert counter.get_total_flops() == 2 * 45 * 256 * 1024
    from torch.overrides import TorchFunctionMode

    class Seen(TorchFunctionMode):
        names = []

        def __torch_function__(self, func, types, args=(), kwargs=None):
            self.names.append(getattr(func, "__name__", ""))
            return func(*args, **(kwargs or {}))
    with Seen():
        ours(a)
    assert "mm" in Seen.names
    traced = torch.jit.trace(ours, (a,), check_trace=False)
    assert torch.equal(traced(2 * a), 2 * want)
    compiled = torch.compile(ours, backend="eager", fullgraph=True)
    assert torch.equal(compiled(a), want)
    with torch.device(DEV):
        assert MM._tiled_takes(a, w, x, None)


def test_project_tells_autograd_that_out_changed():
    """A tensor that autograd saved and project() then overwrote is noticed, and
    inference tensors are written in inference mode only, as by torch's product
    (above the skinny kernel's batch sizes)."""
    from paper_2606_09061_amd import model as MM
    a, w, x = _torch_operands()
    leaf = torch.ones(45, 256, device=DEV, requires_grad=True)
    loss = (leaf * x).sum()             # saves x
    before = x._version
    MM.project(a, w, x)
    assert x._version == before + 1
    with pytest.raises(RuntimeError, match="modified by an inplace operation"):
        loss.backward()
    with torch.inference_mode():
        y = torch.empty(45, 256, dtype=torch.bfloat16, device=DEV)
        MM.project(a, w, y)
        assert torch.equal(y, x)
        before = x._version
        MM.project(a, w, x)
    assert x._version == before + 1
    with pytest.raises(RuntimeError, match="inference"):
        MM.project(a, w, y)


def test_project_attn_of_few_rows_takes_any_workspace():
    """Up to 32 rows, as before the tiled kernel took some of them, a workspace
    that it cannot use does not matter."""
    a, w = _bf16((20, 12288), 67).to(DEV), _bf16((4096, 12288), 68, 0.05).to(DEV)
    out = torch.empty(20, 4096, dtype=torch.bfloat16, device=DEV)
    ws = torch.empty(1 << 24, dtype=torch.uint8, device=DEV)[8:]
    M.project_attn(a, w, out, ws=ws)
    torch.cuda.synchronize()
    want = _f64(a) @ _f64(w).T
    slack = 2.0 ** -20 * (np.abs(_f64(a)) @ np.abs(_f64(w)).T)
    assert np.all(np.abs(_f64(out) - want) <= 2.0 ** -8 * np.abs(want) + slack + 1e-6)


def _small_model():
    cfg = M.ModelConfig(hidden=256, layers=1, hq=4, hkv=2, head_dim=64, inter=512, vocab=1000,
                        theta=1e4)
    return M.Model(cfg, max_seqs=4, max_seq_len=256, max_tokens=256, seed=3, lm_head=True)


@pytest.mark.parametrize("rows", [
    [[1, 40, 1, 41], [0, 0, 70, 70], [2, 100, 33, 133], [3, 0, 1, 1]],   # 105 tokens: tiled GEMMs
    [[1, 40, 1, 41], [0, 0, 20, 20], [2, 100, 5, 105], [3, 0, 1, 1]],    # 27 tokens: skinny and tiled
])
def test_decoder_layer_matches_reference(rows):
    m = _small_model()
    c = m.cfg
    # prior context of slots 1 and 2 already in the pool; slot 0 starts fresh
    rows = np.array(rows, np.int32)
    bt = m.bt.cpu().numpy()
    B = c.block_size
    g = torch.Generator(device="cpu").manual_seed(11)
    prior_k, prior_v = {}, {}
    kc, vc = m.kc[0], m.vc[0]
    kc.fill_(float("nan"))
    vc.fill_(float("nan"))
    for slot, start, _, _ in rows.tolist():
        pk = torch.randn(start, c.hkv, c.head_dim, generator=g).to(torch.bfloat16)
        pv = torch.randn(start, c.hkv, c.head_dim, generator=g).to(torch.bfloat16)
        for p in range(start):
            blk = int(bt[slot, p // B])
            kc[blk, :, p % B, :] = pk[p].to(DEV)
            vc[blk, :, :, p % B] = pv[p].to(DEV)
        prior_k[slot], prior_v[slot] = _f64(pk), _f64(pv)
    T = int(rows[:, 2].sum())
    x0 = _f64(m.embed[m.tokens[:T]])
    L = m.layers[0]
    wts = {k: _f64(v) for k, v in L.items()}
    want, want_k, want_v = ref.decoder_layer(x0, wts, rows.tolist(), prior_k, prior_v, c.hq,
                                             c.hkv, c.head_dim, c.theta, c.eps,
                                             1.0 / math.sqrt(c.head_dim))
    m.forward(rows)
    torch.cuda.synchronize()
    got = _f64(m.x[:T])
    rms = float(np.sqrt((want ** 2).mean()))
    err = np.abs(got - want)
    print(f"layer: rms {rms:.3e} max err {err.max():.3e} mean err {err.mean():.3e}", flush=True)
    assert np.isfinite(got).all()
    assert err.max() <= 0.04 * rms and err.mean() <= 0.006 * rms
    # the new keys and values landed in the pool at their positions (same
    # rounding chain as the output: RMSNorm, GEMM, per-head norm and rotation)
    got_k, got_v = [], []
    for slot, start, length, _ in rows.tolist():
        for j in range(length):
            p = start + j
            blk = int(bt[slot, p // B])
            got_k.append(_f64(kc[blk, :, p % B, :]))
            got_v.append(_f64(vc[blk, :, :, p % B]))
    for got_kv, want_kv in ((np.array(got_k), want_k), (np.array(got_v), want_v)):
        rms_kv = float(np.sqrt((want_kv ** 2).mean()))
        e = np.abs(got_kv - want_kv)
        assert e.max() <= 0.04 * rms_kv and e.mean() <= 0.006 * rms_kv


def test_model_forward_is_deterministic_and_finite(monkeypatch):
    cfg = M.ModelConfig(hidden=256, layers=3, hq=4, hkv=2, head_dim=64, inter=512, vocab=1000)
    m = M.Model(cfg, max_seqs=4, max_seq_len=256, max_tokens=256, seed=5)
    # an iteration plans its batch once: the size is asked for only when the
    # workspace reported too small
    sized = []
    real = M.cp.workspace_bytes
    monkeypatch.setattr(M.cp, "workspace_bytes", lambda d, r: sized.append(1) or real(d, r))
    m.ws = torch.empty(1, dtype=torch.uint8, device=m.dev)   # too small for any plan
    rows1 = np.array([[0, 0, 20, 20], [1, 0, 5, 5]], np.int32)
    t1 = m.forward(rows1)
    assert len(sized) == 1 and m.ws.numel() >= 256
    rows2 = np.array([[0, 20, 1, 21], [1, 5, 1, 6]], np.int32)
    t2 = m.forward(rows2)
    x2 = m.x[:2].clone()
    m.forward(rows1)          # same prefix again, then the same decode step
    t2b = m.forward(rows2)
    torch.cuda.synchronize()
    assert t1.shape == (2,) and t2.shape == (2,)
    assert len(sized) == 1, "a later iteration planned twice"
    assert torch.equal(t2, t2b) and torch.equal(x2, m.x[:2])
    assert torch.isfinite(m.x[:2].float()).all()


@pytest.mark.parametrize("M,N,K", [(1, 32, 256), (17, 96, 512), (32, 4096, 4096), (33, 64, 256),
                                   (64, 6144, 4096), (100, 4096, 12288), (128, 1024, 1024),
                                   (70, 64, 768), (5, 160, 1280), (9, 4096, 12288),
                                   (1, 1024, 512)])
@pytest.mark.parametrize("residual", [False, True])
def test_gemm_skinny_matches_reference(M, N, K, residual):
    print(f"gemm_skinny M={M} N={N} K={K} residual={residual}", flush=True)
    a = _bf16((M, K), 21)
    w = _bf16((N, K), 22, 0.05)
    r = _bf16((M, N), 23) if residual else None
    out = (r.clone() if residual else torch.empty(M, N, dtype=torch.bfloat16)).to(DEV)
    ad, wd = a.to(DEV), w.to(DEV)
    from paper_2606_09061_amd import model as MM
    MM.gemm_skinny(ad, wd, out, out if residual else None)
    torch.cuda.synchronize()
    want = _f64(a) @ _f64(w).T + (_f64(r) if residual else 0.0)
    # fp32 accumulation over K terms, then one bf16 rounding
    slack = 2.0 ** -20 * (np.abs(_f64(a)) @ np.abs(_f64(w)).T)
    err = np.abs(_f64(out) - want)
    assert np.all(err <= 2.0 ** -8 * np.abs(want) + slack + 1e-6), f"max err {err.max():.3e}"


def test_gemm_skinny_rejects_unsupported_shapes():
    lib = M.load()
    x = torch.zeros(256, 256, dtype=torch.bfloat16, device=DEV)
    p = x.data_ptr()
    assert lib.cpl_gemm_skinny(p, p + 16 * 256 * 2, None, p + 64 * 256 * 2, 129, 32, 256, None) != 0
    assert lib.cpl_gemm_skinny(p, p, None, p + 1024, 8, 48, 256, None) != 0     # N % 32
    assert lib.cpl_gemm_skinny(p, p, None, p + 1024, 8, 32, 320, None) != 0    # K % 256
    assert lib.cpl_gemm_skinny(p, p, None, p, 8, 32, 256, None) != 0           # a aliases c


@pytest.mark.parametrize("M,N,K", [(1, 128, 32), (33, 256, 64), (64, 384, 4096), (65, 128, 96),
                                   (130, 6144, 4096), (257, 4096, 4096), (1000, 512, 1024),
                                   (128, 1024, 1024), (4096, 256, 128), (200, 24576, 64)])
@pytest.mark.parametrize("residual", ["none", "separate", "in_place"])
@pytest.mark.parametrize("split", ["auto", "none"])
def test_gemm_matches_reference(monkeypatch, M, N, K, residual, split):
    """cpl_gemm against the fp64 product of the same bf16 inputs: ragged row
    counts (tiles past M), one and many K stages, the layer's QKV (N 6144) and
    output (N 4096) shapes, residual read from another tensor or from the
    output itself; K split into slices summed by a second kernel (auto) or
    not split."""
    print(f"gemm M={M} N={N} K={K} residual={residual} split={split}", flush=True)
    if split == "none":
        monkeypatch.setenv("CPL_GEMM_SPLIT", "1")
    from paper_2606_09061_amd import model as MM
    a = _bf16((M, K), 41)
    w = _bf16((N, K), 42, 0.05)
    r = _bf16((M, N), 43) if residual != "none" else None
    ad, wd = a.to(DEV), w.to(DEV)
    if residual == "in_place":
        out = r.clone().to(DEV)
        MM.gemm(ad, wd, out, out)
    else:
        out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=DEV)
        MM.gemm(ad, wd, out, r.to(DEV) if r is not None else None)
    torch.cuda.synchronize()
    want = _f64(a) @ _f64(w).T + (_f64(r) if r is not None else 0.0)
    slack = 2.0 ** -20 * (np.abs(_f64(a)) @ np.abs(_f64(w)).T)
    got = _f64(out)
    assert np.isfinite(got).all()
    err = np.abs(got - want)
    assert np.all(err <= 2.0 ** -8 * np.abs(want) + slack + 1e-6), f"max err {err.max():.3e}"


@pytest.mark.parametrize("M,N,K,split", [
    (1, 768, 64, 1),       # one row, fewer stages than ring slots
    (45, 768, 1088, 3),    # odd stage count, uneven slices
    (301, 768, 448, 1),    # ragged last row block
    (577, 768, 128, 2),    # several row groups, one stage per slice
    (130, 256, 416, 2),    # K an odd number of 32s, split
])
@pytest.mark.parametrize("cfg", range(17))
def test_gemm_every_tile_matches_reference(monkeypatch, cfg, M, N, K, split):
    """Each tile configuration of cpl_gemm (768 columns divide into all of
    them), against the fp64 product; the bound is test_gemm_matches_reference's."""
    if K % 64 and cfg:
        pytest.skip("one kernel takes these K, whatever the configuration")
    print(f"gemm cfg={cfg} M={M} N={N} K={K} split={split}", flush=True)
    monkeypatch.setenv("CPL_GEMM_CFG", str(cfg))
    monkeypatch.setenv("CPL_GEMM_SPLIT", str(split))
    from paper_2606_09061_amd import model as MM
    a, w, r = _bf16((M, K), 51), _bf16((N, K), 52, 0.05), _bf16((M, N), 53)
    out = r.clone().to(DEV)
    MM.gemm(a.to(DEV), w.to(DEV), out, out)
    torch.cuda.synchronize()
    want = _f64(a) @ _f64(w).T + _f64(r)
    slack = 2.0 ** -20 * (np.abs(_f64(a)) @ np.abs(_f64(w)).T)
    err = np.abs(_f64(out) - want)
    assert np.all(err <= 2.0 ** -8 * np.abs(want) + slack + 1e-6), f"max err {err.max():.3e}"


def _gemm_error_on_gpu(M, N, K, residual):
    """cpl_gemm's largest excess over test_gemm_matches_reference's bound, and
    whether every result is finite; the fp64 products by columns on the GPU."""
    from paper_2606_09061_amd import model as MM
    g = torch.Generator(device=DEV).manual_seed(M + N + K)

    def randn(*shape, scale=1.0):
        return (torch.randn(*shape, generator=g, device=DEV) * scale).to(torch.bfloat16)
    a, w, r = randn(M, K), randn(N, K, scale=0.05), randn(M, N)
    out = r.clone() if residual else torch.full_like(r, float("nan"))
    MM.gemm(a, w, out, out if residual else None)
    excess = -math.inf
    ad = a.double()
    for n in range(0, N, 8192):
        wd = w[n:n + 8192].double().t().contiguous()
        want = ad @ wd + (r[:, n:n + 8192].double() if residual else 0.0)
        bound = 2.0 ** -8 * want.abs() + 2.0 ** -20 * (ad.abs() @ wd.abs()) + 1e-6
        excess = max(excess, float(((out[:, n:n + 8192].double() - want).abs() - bound).max()))
    return excess, bool(torch.isfinite(out.float()).all())


@pytest.mark.parametrize("M,N,K,residual", [
    (24, 24576, 4096, False), (96, 24576, 4096, False), (261, 24576, 4096, False),
    (300, 28672, 2048, False),
    (45, 4096, 12288, True), (261, 4096, 12288, True),
    (24, 151936, 512, False), (65, 151936, 512, True),   # more than two tiles per CU
])
def test_gemm_of_large_weights_matches_reference(M, N, K, residual):
    """The forms that weights of 32 M elements and more take: copies that bypass
    the caches in both kernels, and XCDs that start at the same stage where
    there are more than two tiles per CU."""
    print(f"gemm of large weights M={M} N={N} K={K}", flush=True)
    excess, finite = _gemm_error_on_gpu(M, N, K, residual)
    assert finite and excess <= 0.0


@pytest.mark.parametrize("M,N,K", [(1, 128, 416), (45, 256, 416), (64, 6144, 2080), (45, 384, 1056),
                                   (130, 256, 1056), (2000, 1024, 2080)])
@pytest.mark.parametrize("split", ["auto", "1", "3"])
def test_gemm_of_half_stages_matches_reference(monkeypatch, M, N, K, split):
    """K an odd number of 32s, many stages long, on both of its tiles."""
    print(f"gemm of half stages M={M} N={N} K={K} split={split}", flush=True)
    if split != "auto":
        monkeypatch.setenv("CPL_GEMM_SPLIT", split)
    excess, finite = _gemm_error_on_gpu(M, N, K, True)
    assert finite and excess <= 0.0


def _zeros_or_skip(*shape):
    if torch.cuda.mem_get_info(DEV)[0] < 1.1 * 2 * math.prod(shape):
        pytest.skip("not enough free GPU memory")
    return torch.zeros(*shape, dtype=torch.bfloat16, device=DEV)


@pytest.mark.parametrize("K", [306783392, 306783424])
def test_gemm_of_rows_beyond_32_bits(K):
    """Eight rows of this many k (a whole and a half last stage) span more than
    4 GiB, the reach of a 32-bit offset from the first of them.  A few columns
    of the operands are not zero, so that the fp64 product is small."""
    print(f"gemm of long rows K={K}", flush=True)
    a, w = _zeros_or_skip(9, K), _zeros_or_skip(128, K)
    cols = torch.tensor([0, 1, 63, 64, 1000003, K // 2, K - 65, K - 33, K - 32, K - 1], device=DEV)
    av, wv = _bf16((9, 10), 71), _bf16((128, 10), 72)
    a[:, cols], w[:, cols] = av.to(DEV), wv.to(DEV)
    out = torch.full((9, 128), float("nan"), dtype=torch.bfloat16, device=DEV)
    M.gemm(a, w, out)
    torch.cuda.synchronize()
    _close(_f64(out), _f64(av) @ _f64(wv).T, abs_=1e-4)
    del a, w
    torch.cuda.empty_cache()


def test_gemm_of_more_columns_than_a_grid_row_holds():
    """2^30 + 128 columns are more workgroups than one row of a launch's grid
    takes.  A few rows of the weights are not zero."""
    N, K = (1 << 30) + 128, 32
    print(f"gemm of many columns N={N}", flush=True)
    w, out = _zeros_or_skip(N, K), _zeros_or_skip(1, N)
    rows = torch.tensor([0, 127, 128, 1 << 20, (1 << 27) - 1, 1 << 27, 1 << 29, N - 129, N - 1],
                        device=DEV)
    a, wv = _bf16((1, K), 73), _bf16((9, K), 74)
    w[rows] = wv.to(DEV)
    out.fill_(float("nan"))
    M.gemm(a.to(DEV), w, out)
    torch.cuda.synchronize()
    _close(_f64(out[:, rows]), _f64(a) @ _f64(wv).T, abs_=1e-4)
    out[:, rows] = 0
    assert int(torch.count_nonzero(out)) == 0
    del w, out
    torch.cuda.empty_cache()


def test_gemm_rejects_unsupported_shapes():
    lib = M.load()
    x = torch.zeros(512, 512, dtype=torch.bfloat16, device=DEV)
    p = x.data_ptr()
    c = p + 256 * 512 * 2
    assert lib.cpl_gemm(p, p, None, c, 0, 128, 32, None, 0, None) != 0        # M = 0
    assert lib.cpl_gemm(p, p, None, c, 8, 96, 32, None, 0, None) != 0         # N % 128
    assert lib.cpl_gemm(p, p, None, c, 8, 128, 48, None, 0, None) != 0        # K % 32
    assert lib.cpl_gemm(p, p, None, p, 8, 128, 32, None, 0, None) != 0        # a aliases c
    assert lib.cpl_gemm(p + 8, p, None, c, 8, 128, 32, None, 0, None) != 0    # misaligned a
    assert lib.cpl_gemm(p, p, None, c, 8, 128, 32, None, 0, None) == 0
    torch.cuda.synchronize()
