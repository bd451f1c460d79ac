"""GPU parity of the PTC preconditioner kernels and of the FGCR / CGNR solvers.

PTC kernels run in FP32 with FP32 accumulation; they are compared with the FP64
oracle fed the same weights (for the BF16 kernels: the same BF16-rounded
weights).  Tolerance 2e-5 relative: FP32 unit roundoff 6e-8 times the ~9 x 8
paths x channels and the 3-term colour / 4-term spin sums of one output.
Solvers are judged by the oracle-restated residual ||b - D x|| / ||b||.
"""

import numpy as np
import pytest
import torch

from oracle import oracle as orc
from oracle import ptc
from paper_1405_0700_amd import synth
from paper_1405_0700_amd import wilson as W

pytestmark = pytest.mark.gpu
AP = (1, 1, 1, -1)
TOL32 = 2e-5


@pytest.fixture(autouse=True)
def _announce(request):
    print("\n[gpu case] %s" % request.node.nodeid, flush=True)
    yield


def rel(a, b):
    a, b = np.asarray(a), np.asarray(b)
    return float(np.linalg.norm((a - b).ravel()) / np.linalg.norm(b.ravel()))


def random_phases(seed):
    rng = np.random.default_rng(seed)
    return tuple(np.exp(1j * rng.uniform(0, 2 * np.pi, 4)))


def random_weights(cout, cin, seed, scale=1.0):
    rng = np.random.default_rng(seed)
    z = rng.standard_normal((9, cout, cin, 4, 4, 2)) * scale
    return z[..., 0] + 1j * z[..., 1]


def dev_weights(w):
    """complex weights -> FP32 device tensor (re, im interleaved) and the FP32-rounded complex copy"""
    f = np.stack([w.real, w.imag], -1).astype(np.float32)
    return torch.as_tensor(np.ascontiguousarray(f)).cuda(), (f[..., 0] + 1j * f[..., 1]).astype(np.complex128)


def bf16_round(w):
    """FP64 -> FP32 -> BF16 (round to nearest even) -> value, per real component"""
    def r(x):
        b = np.ascontiguousarray(x.astype(np.float32)).view(np.uint32).astype(np.uint64)
        b = ((b + 0x7FFF + ((b >> 16) & 1)) >> 16) << 16
        return b.astype(np.uint32).view(np.float32).astype(np.float64)
    return r(w.real) + 1j * r(w.imag)


def f32(x):
    return np.asarray(x).astype(np.complex64).astype(np.complex128)


_cache = {}


def lattice(dims, seed, phases=AP, eps=0.5):
    key = (dims, seed, phases, eps)
    if key not in _cache:
        u = synth.su3_links(dims, eps, seed)
        _cache[key] = (u, W.Lattice.create(u, phases))
    return _cache[key]


def channels(lat, fields):
    """list of canonical fields -> internal channel-major FP32 field (one FULL field per channel)"""
    return torch.cat([lat.pack(f32(f), W.WL_FULL, W.WL_F32) for f in fields])


def unchannels(lat, internal, n, dims):
    lx, ly, lz, lt = dims
    per = internal.numel() // n
    return [lat.unpack(internal[k * per:(k + 1) * per], W.WL_FULL, W.WL_F32).reshape(lt, lz, ly, lx, 4, 3)
            for k in range(n)]


DIMS = (4, 6, 4, 8)


@pytest.mark.parametrize("cout,cin", [(8, 1), (1, 8), (3, 2)])
def test_layer_forward_and_adjoint(cout, cin):
    ph = random_phases(1)
    u, lat = lattice(DIMS, 2, ph)
    w = random_weights(cout, cin, 3, 0.3)
    wd, w32 = dev_weights(w)
    ins = [synth.gaussian_spinor(DIMS, seed=10 + b) for b in range(cin)]
    out = torch.cat([lat.new(W.WL_FULL, W.WL_F32) for _ in range(cout)])
    W.wl_ptc_layer(lat.ctx, out, channels(lat, ins), wd, cout, cin)
    want = ptc.layer([f32(f) for f in ins], w32, u, ph)
    got = unchannels(lat, out, cout, DIMS)
    assert rel(np.stack(got), np.stack(want)) < TOL32
    # adjoint: cout_f = cout, cin_f = cin; the adjoint launch maps cout -> cin channels
    gs = [synth.gaussian_spinor(DIMS, seed=20 + a) for a in range(cout)]
    gin = torch.cat([lat.new(W.WL_FULL, W.WL_F32) for _ in range(cin)])
    W.wl_ptc_layer(lat.ctx, gin, channels(lat, gs), wd, cin, cout, adjoint=True)
    want = ptc.layer_adjoint([f32(g) for g in gs], w32, u, ph)
    assert rel(np.stack(unchannels(lat, gin, cin, DIMS)), np.stack(want)) < TOL32


@pytest.mark.parametrize("cout,cin", [(8, 1), (1, 8)])
def test_weight_gradient(cout, cin):
    ph = random_phases(4)
    u, lat = lattice(DIMS, 5, ph)
    gs = [synth.gaussian_spinor(DIMS, seed=30 + a) for a in range(cout)]
    ins = [synth.gaussian_spinor(DIMS, seed=40 + b) for b in range(cin)]
    grad = torch.zeros((9, cout, cin, 4, 4, 2), dtype=torch.float64, device="cuda")
    W.wl_ptc_weight_grad(lat.ctx, grad, channels(lat, gs), channels(lat, ins), cout, cin)
    W.wl_ptc_weight_grad(lat.ctx, grad, channels(lat, gs), channels(lat, ins), cout, cin, accumulate=True)
    torch.cuda.synchronize()
    g = grad.cpu().numpy()
    got = g[..., 0] + 1j * g[..., 1]
    want = ptc.weight_grad([f32(x) for x in gs], [f32(x) for x in ins], u, ph)
    assert rel(got, 2 * want) < TOL32


def test_special_weights_give_the_hopping_term():
    ph = random_phases(6)
    u, lat = lattice(DIMS, 7, ph)
    w = np.zeros((9, 1, 1, 4, 4), dtype=np.complex128)
    for mu in range(4):
        g = orc.gamma(mu)
        w[1 + 2 * mu, 0, 0] = np.eye(4) - g
        w[2 + 2 * mu, 0, 0] = np.eye(4) + g
    wd, _ = dev_weights(w)
    phi = synth.gaussian_spinor(DIMS, seed=8)
    out = lat.new(W.WL_FULL, W.WL_F32)
    W.wl_ptc_layer(lat.ctx, out, channels(lat, [phi]), wd, 1, 1)
    h = lat.new(W.WL_FULL, W.WL_F32)
    W.wl_dslash_apply(lat.ctx, h, lat.pack(phi, W.WL_FULL, W.WL_F32), W.WL_FULL, W.WL_F32, 18)
    want = orc.hop(phi, u, ph)
    got = unchannels(lat, out, 1, DIMS)[0]
    assert rel(got, want) < TOL32
    assert rel(got, lat.unpack(h, W.WL_FULL, W.WL_F32).reshape(want.shape)) < TOL32


def test_network_apply_uses_bf16_weights():
    ph = random_phases(9)
    u, lat = lattice(DIMS, 10, ph)
    w1, w2 = synth.ptc_weights(8, seed=530)
    w1 = w1 + random_weights(8, 1, 11, 0.05)
    net = W.wl_ptc_create(w1, w2)
    r = synth.gaussian_spinor(DIMS, seed=12)
    out = lat.new(W.WL_FULL, W.WL_F32)
    W.wl_ptc_apply(lat.ctx, net, out, channels(lat, [r]))
    want, _ = ptc.net_apply(f32(r), bf16_round(w1), bf16_round(w2), u, ph)
    assert rel(unchannels(lat, out, 1, DIMS)[0], want) < TOL32
    W.wl_ptc_destroy(net)


def test_training_gradients_loss_and_adam_step():
    ph = random_phases(13)
    u, lat = lattice(DIMS, 14, ph)
    w1, w2 = synth.ptc_weights(4, seed=15)
    w1 = w1 + random_weights(4, 1, 16, 0.05)
    w2 = w2 + random_weights(1, 4, 17, 0.05)
    net = W.wl_ptc_create(w1, w2)
    pairs = [(synth.gaussian_spinor(DIMS, seed=20 + i), synth.gaussian_spinor(DIMS, seed=30 + i)) for i in range(3)]
    for r, e in pairs:
        W.wl_ptc_accumulate(lat.ctx, net, channels(lat, [r]), channels(lat, [e]), 1.0 / len(pairs))
    g1, g2 = W.wl_ptc_get_grads(net, 4)
    w1b, w2b = bf16_round(w1), bf16_round(w2)
    loss_o, g1o, g2o = ptc.loss_and_grads([(f32(r), f32(e)) for r, e in pairs], w1b, w2b, u, ph)
    assert rel(g1, g1o) < 1e-4 and rel(g2, g2o) < 1e-4
    m1, m2 = W.wl_ptc_get_weights(net, 4)
    loss = W.wl_ptc_step(net, 1e-3)
    assert abs(loss - loss_o) < 1e-5 * loss_o
    n1, n2 = W.wl_ptc_get_weights(net, 4)
    # first Adam step: every real parameter with a non-negligible gradient moves by lr against its sign
    for w_old, w_new, g in ((m1, n1, g1o), (m2, n2, g2o)):
        d = w_new - w_old
        big = np.abs(g.real) > 1e-3 * np.abs(g).max()
        assert np.allclose(d.real[big], -1e-3 * np.sign(g.real[big]), atol=2e-6)
        big = np.abs(g.imag) > 1e-3 * np.abs(g).max()
        assert np.allclose(d.imag[big], -1e-3 * np.sign(g.imag[big]), atol=2e-6)
    # gradients were cleared by the step
    c1, c2 = W.wl_ptc_get_grads(net, 4)
    assert not np.any(c1) and not np.any(c2)
    W.wl_ptc_destroy(net)


def test_residual_loss_gradients():
    ph = random_phases(18)
    u, lat = lattice(DIMS, 19, ph)
    kappa = 0.12
    w1, w2 = synth.ptc_weights(4, seed=21)
    w1 = w1 + random_weights(4, 1, 22, 0.05)
    w2 = w2 + random_weights(1, 4, 23, 0.05)
    net = W.wl_ptc_create(w1, w2)
    rs = [synth.gaussian_spinor(DIMS, seed=40 + i) for i in range(2)]
    for r in rs:
        W.wl_ptc_accumulate_residual(lat.ctx, net, channels(lat, [r]), kappa, 1.0 / len(rs))
    g1, g2 = W.wl_ptc_get_grads(net, 4)
    loss_o, g1o, g2o = ptc.loss_and_grads_residual([f32(r) for r in rs], bf16_round(w1), bf16_round(w2), u, ph, kappa)
    assert rel(g1, g1o) < 1e-4 and rel(g2, g2o) < 1e-4
    loss = W.wl_ptc_step(net, 1e-3)
    assert abs(loss - loss_o) < 1e-5 * loss_o
    W.wl_ptc_destroy(net)


# ------------------------------------------------------------------ solvers
def system_resid(u, kappa, x, b):
    return float(np.linalg.norm(orc.dirac(x, u, kappa, AP) - b) / np.linalg.norm(b))


@pytest.mark.parametrize("use_net", [False, True])
def test_fgcr_solves_the_system(use_net):
    dims = (4, 4, 4, 8)
    kappa = 0.12
    u, lat = lattice(dims, 50, AP)
    b = synth.gaussian_spinor(dims, seed=51)
    net = W.wl_ptc_create(*synth.ptc_weights(8, seed=530)) if use_net else None
    x = lat.new(W.WL_FULL)
    p = W.wl_fgcr_params_default()
    p.fallback = 0
    st, info = W.wl_fgcr_solve(lat.ctx, x, lat.pack(b), kappa, net, p)
    r = system_resid(u, kappa, lat.unpack(x).reshape(b.shape), b)
    print("net", use_net, info, "oracle residual", r)
    assert st == W.WL_OK and info["fallback"] == 0
    assert r <= 1.05e-10
    if net:
        W.wl_ptc_destroy(net)


def test_cgnr_stops_on_the_system_residual():
    dims = (4, 4, 4, 8)
    kappa = 0.12
    u, lat = lattice(dims, 52, AP)
    b = synth.gaussian_spinor(dims, seed=53)
    x = lat.new(W.WL_FULL)
    st, info = W.wl_cgnr_solve(lat.ctx, x, lat.pack(b), kappa)
    r = system_resid(u, kappa, lat.unpack(x).reshape(b.shape), b)
    assert st == W.WL_OK and r <= 1.05e-10 and info["true_rel_resid"] <= 1e-10


def test_fgcr_falls_back_to_cg_on_a_broken_network():
    dims = (4, 4, 4, 8)
    kappa = 0.12
    u, lat = lattice(dims, 54, AP)
    b = synth.gaussian_spinor(dims, seed=55)
    zero = np.zeros((9, 4, 1, 4, 4), dtype=np.complex128)
    net = W.wl_ptc_create(zero, np.zeros((9, 1, 4, 4, 4), dtype=np.complex128))  # M = 0
    x = lat.new(W.WL_FULL)
    st, info = W.wl_fgcr_solve(lat.ctx, x, lat.pack(b), kappa, net)
    r = system_resid(u, kappa, lat.unpack(x).reshape(b.shape), b)
    assert st == W.WL_OK and info["fallback"] == 1 and info["fallback_iters"] > 0
    assert r <= 1.05e-10
    p = W.wl_fgcr_params_default()
    p.fallback = 0
    st, info = W.wl_fgcr_solve(lat.ctx, lat.new(W.WL_FULL), lat.pack(b), kappa, net, p)
    assert st == W.WL_NOT_CONVERGED and info["fallback"] == 0
    W.wl_ptc_destroy(net)


@pytest.mark.parametrize("use_net", [False, True])
@pytest.mark.parametrize("dims,kappa,eps", [((4, 4, 4, 8), 0.12, 0.5), ((8, 8, 8, 8), 0.137, 0.2)])
def test_preconditioned_cgnr_solves_the_system(use_net, dims, kappa, eps):
    """CG on the normal equations of D M: converges also at kappa = 0.137 with eps = 0.2
    links, where D's spectrum surrounds the origin (restarted GCR stalls there)."""
    u, lat = lattice(dims, 56, AP, eps)
    b = synth.gaussian_spinor(dims, seed=57)
    w1, w2 = synth.ptc_weights(8, seed=530)
    net = W.wl_ptc_create(w1, w2) if use_net else None
    x = lat.new(W.WL_FULL)
    p = W.wl_pcgnr_params_default()
    p.fallback = 0
    st, info = W.wl_pcgnr_solve(lat.ctx, x, lat.pack(b), kappa, net, p)
    r = system_resid(u, kappa, lat.unpack(x).reshape(b.shape), b)
    print("net", use_net, info, "oracle residual", r)
    assert st == W.WL_OK and info["fallback"] == 0 and info["restarts"] >= 2
    assert r <= 1.05e-10 and info["true_rel_resid"] <= 1e-10
    if net:
        W.wl_ptc_destroy(net)


def test_preconditioned_cgnr_zero_source_and_bad_parameters():
    u, lat = lattice((4, 4, 4, 8), 58, AP)
    x = lat.pack(synth.gaussian_spinor((4, 4, 4, 8), seed=59))
    st, info = W.wl_pcgnr_solve(lat.ctx, x, lat.new(W.WL_FULL), 0.12)
    assert st == W.WL_OK and not torch.any(x != 0)
    p = W.wl_pcgnr_params_default()
    p.inner_tol = 1.5
    with pytest.raises(W.WilsonError):
        W.wl_pcgnr_solve(lat.ctx, lat.new(W.WL_FULL), lat.pack(synth.gaussian_spinor((4, 4, 4, 8), seed=60)), 0.12,
                         None, p)


def test_adam_steps_match_oracle():
    """Six Adam steps: the GPU's FP32 master weights and both moments follow repeated calls of the
    oracle's adam_step fed the gradients the GPU accumulated at each step (so the moments' carry-over
    and the bias corrections at t = 1 .. 6 are pinned, not only the first step's sign rule); each
    step's gradient is also checked against the oracle's gradient at the GPU's current BF16 weights."""
    ph = random_phases(61)
    u, lat = lattice(DIMS, 62, ph)
    w1, w2 = synth.ptc_weights(4, seed=63)
    w1 = w1 + random_weights(4, 1, 64, 0.05)
    w2 = w2 + random_weights(1, 4, 65, 0.05)
    net = W.wl_ptc_create(w1, w2)
    pairs = [(synth.gaussian_spinor(DIMS, seed=70 + i), synth.gaussian_spinor(DIMS, seed=80 + i)) for i in range(2)]
    ins = [(channels(lat, [r]), channels(lat, [e])) for r, e in pairs]
    ow1, ow2 = W.wl_ptc_get_weights(net, 4)  # the FP32 master weights the steps start from
    om1 = np.zeros(ow1.shape + (2,))
    om2 = np.zeros(ow2.shape + (2,))
    ov1, ov2 = np.zeros_like(om1), np.zeros_like(om2)
    lr = 2e-3
    for t in range(1, 7):
        for r, e in ins:
            W.wl_ptc_accumulate(lat.ctx, net, r, e, 1.0 / len(ins))
        g1, g2 = W.wl_ptc_get_grads(net, 4)
        cw1, cw2 = W.wl_ptc_get_weights(net, 4)
        _, g1o, g2o = ptc.loss_and_grads([(f32(r), f32(e)) for r, e in pairs], bf16_round(cw1), bf16_round(cw2), u,
                                         ph)
        assert rel(g1, g1o) < 1e-4 and rel(g2, g2o) < 1e-4, t
        W.wl_ptc_step(net, lr)
        ow1, om1, ov1 = ptc.adam_step(ow1, g1, om1, ov1, t, lr=lr)
        ow2, om2, ov2 = ptc.adam_step(ow2, g2, om2, ov2, t, lr=lr)
        n1, n2 = W.wl_ptc_get_weights(net, 4)
        m1, m2, v1, v2 = W.wl_ptc_get_moments(net, 4)
        # FP32 state against the FP64 restatement: moments to a few FP32 roundings; the weights move by
        # at most lr per step, so their difference is judged against lr
        assert rel(m1, om1) < 1e-5 and rel(m2, om2) < 1e-5, t
        assert rel(v1, ov1) < 1e-5 and rel(v2, ov2) < 1e-5, t
        assert np.abs(n1 - ow1).max() < 1e-3 * lr and np.abs(n2 - ow2).max() < 1e-3 * lr, t
    W.wl_ptc_destroy(net)


@pytest.mark.parametrize("adjoint", [False, True])
def test_network_on_several_rhs(adjoint):
    """M (and M^+) on a FULL field of 3 right-hand sides equals the one-rhs application of each, bit for bit
    (the same arithmetic per point), and the oracle's network (its adjoint: the two layer adjoints in reverse
    order) within the FP32 tolerance."""
    ph = random_phases(91)
    u, lat = lattice(DIMS, 92, ph)
    w1, w2 = synth.ptc_weights(4, seed=93)
    w1 = w1 + random_weights(4, 1, 94, 0.05)
    w2 = w2 + random_weights(1, 4, 95, 0.05)
    net = W.wl_ptc_create(w1, w2)
    fields = [f32(synth.gaussian_spinor(DIMS, seed=96 + r)) for r in range(3)]
    stack = np.stack([f.reshape(-1, 4, 3) for f in fields])
    out = lat.new(W.WL_FULL, W.WL_F32, 3)
    W.wl_ptc_apply(lat.ctx, net, out, lat.pack(stack, W.WL_FULL, W.WL_F32, 3), nrhs=3, adjoint=adjoint)
    multi = lat.unpack(out, W.WL_FULL, W.WL_F32, 3)
    w1b, w2b = bf16_round(w1), bf16_round(w2)
    for r, f in enumerate(fields):
        o1 = lat.new(W.WL_FULL, W.WL_F32)
        W.wl_ptc_apply(lat.ctx, net, o1, lat.pack(f, W.WL_FULL, W.WL_F32), adjoint=adjoint)
        assert np.array_equal(multi[r], lat.unpack(o1, W.WL_FULL, W.WL_F32))
        if adjoint:
            hidden = ptc.layer_adjoint([f], w2b, u, ph)
            want = ptc.layer_adjoint(hidden, w1b, u, ph)[0]
        else:
            want, _ = ptc.net_apply(f, w1b, w2b, u, ph)
        assert rel(multi[r].reshape(want.shape), want) < TOL32
    W.wl_ptc_destroy(net)


def test_cgnr_and_preconditioned_cgnr_on_several_rhs():
    """Four right-hand sides in one solve (kappa 0.137, eps 0.2 links on 8^4, where D's spectrum surrounds
    the origin): plain FP64 CGNR and CG on the normal equations of D M (network and M = 1) bring every rhs
    to an oracle-restated system residual <= 1e-10; the multi-rhs iteration counts stay within a few of the
    one-rhs solves of the same sources (the same arithmetic per point; only the reductions' order differs)."""
    dims, kappa = (8, 8, 8, 8), 0.137
    u, lat = lattice(dims, 97, AP, 0.2)
    srcs = [synth.gaussian_spinor(dims, seed=98 + r) for r in range(4)]
    stack = np.stack([s.reshape(-1, 4, 3) for s in srcs])
    B = lat.pack(stack, W.WL_FULL, W.WL_F64, 4)
    w1, w2 = synth.ptc_weights(8, seed=530)
    net = W.wl_ptc_create(w1, w2)
    x = lat.new(W.WL_FULL, W.WL_F64, 4)
    st, infos = W.wl_cgnr_solve(lat.ctx, x, B, kappa, nrhs=4)
    xs = lat.unpack(x, W.WL_FULL, W.WL_F64, 4)
    assert st == W.WL_OK
    for r in range(4):
        assert system_resid(u, kappa, xs[r].reshape(srcs[r].shape), srcs[r]) <= 1.05e-10
    for m in (None, net):
        x = lat.new(W.WL_FULL, W.WL_F64, 4)
        p = W.wl_pcgnr_params_default()
        p.fallback = 0
        st, infos = W.wl_pcgnr_solve(lat.ctx, x, B, kappa, m, p, nrhs=4)
        xs = lat.unpack(x, W.WL_FULL, W.WL_F64, 4)
        assert st == W.WL_OK
        for r in range(4):
            res = system_resid(u, kappa, xs[r].reshape(srcs[r].shape), srcs[r])
            x1 = lat.new(W.WL_FULL)
            st1, one = W.wl_pcgnr_solve(lat.ctx, x1, lat.pack(srcs[r]), kappa, m, p)
            print("net", m is not None, "rhs", r, infos[r], "oracle", res, "one-rhs iters", one["iters"])
            assert res <= 1.05e-10 and infos[r]["true_rel_resid"] <= 1e-10 and infos[r]["fallback"] == 0
            assert abs(infos[r]["iters"] - one["iters"]) <= max(3, one["iters"] // 20)
    W.wl_ptc_destroy(net)


@pytest.mark.parametrize("channels,nrhs,adjoint", [(8, 1, False), (8, 3, True), (4, 3, False), (4, 1, True),
                                                   (8, 5, False), (6, 2, False), (6, 2, True)])
def test_network_on_matrix_cores(channels, nrhs, adjoint):
    """M (M^+) through the matrix-core network kernel (4 or 8 channels; 6 takes the layer kernels) against the
    oracle's two layers (their adjoints in reverse order) with the same BF16 weights.  6x6x2x2 has V/2 = 72
    points per parity, so every nrhs leaves a partial last tile of 16 points."""
    dims = (6, 6, 2, 2)
    ph = random_phases(600 + channels)
    u, lat = lattice(dims, 601, ph)
    w1, w2 = synth.ptc_weights(channels, seed=602)
    w1 = w1 + random_weights(channels, 1, 603, 0.05)
    w2 = w2 + random_weights(1, channels, 604, 0.05)
    net = W.wl_ptc_create(w1, w2)
    fields = [f32(synth.gaussian_spinor(dims, seed=610 + r)) for r in range(nrhs)]
    stack = np.stack([f.reshape(-1, 4, 3) for f in fields])
    out = lat.new(W.WL_FULL, W.WL_F32, nrhs)
    W.wl_ptc_apply(lat.ctx, net, out, lat.pack(stack, W.WL_FULL, W.WL_F32, nrhs), nrhs=nrhs, adjoint=adjoint)
    got = lat.unpack(out, W.WL_FULL, W.WL_F32, nrhs)
    w1b, w2b = bf16_round(w1), bf16_round(w2)
    for r, f in enumerate(fields):
        if adjoint:
            want = ptc.layer_adjoint(ptc.layer_adjoint([f], w2b, u, ph), w1b, u, ph)[0]
        else:
            want, _ = ptc.net_apply(f, w1b, w2b, u, ph)
        g = (got[r] if nrhs > 1 else got).reshape(want.shape)
        assert rel(g, want) < TOL32, (r, rel(g, want))
        assert np.abs(g - want).max() < TOL32 * np.abs(want).max()
    W.wl_ptc_destroy(net)


@pytest.mark.parametrize("channels,nrhs,dims", [(8, 3, (12, 10, 14, 22)), (3, 1, (24, 18, 20, 22))])
def test_network_where_waves_take_several_tiles(channels, nrhs, dims):
    """More tiles of 16 points than resident waves (3,072 for 8 channels, 4,096 for up to 4), ranges that do not
    divide evenly over XCDs and a partial last tile: every point of the last right-hand side against the oracle."""
    ph = random_phases(640 + channels)
    u, lat = lattice(dims, 641, ph)
    w1, w2 = synth.ptc_weights(channels, seed=642)
    w1 = w1 + random_weights(channels, 1, 643, 0.05)
    w2 = w2 + random_weights(1, channels, 644, 0.05)
    net = W.wl_ptc_create(w1, w2)
    fields = [f32(synth.gaussian_spinor(dims, seed=650 + r)) for r in range(nrhs)]
    stack = np.stack([f.reshape(-1, 4, 3) for f in fields])
    out = lat.new(W.WL_FULL, W.WL_F32, nrhs)
    W.wl_ptc_apply(lat.ctx, net, out, lat.pack(stack, W.WL_FULL, W.WL_F32, nrhs), nrhs=nrhs)
    got = lat.unpack(out, W.WL_FULL, W.WL_F32, nrhs)
    want, _ = ptc.net_apply(fields[-1], bf16_round(w1), bf16_round(w2), u, ph)
    g = (got[-1] if nrhs > 1 else got).reshape(want.shape)
    assert rel(g, want) < TOL32
    assert np.abs(g - want).max() < TOL32 * np.abs(want).max()
    W.wl_ptc_destroy(net)


def test_network_tables_follow_the_weights():
    """After an Adam step the matrix-core network uses the new BF16 weights (its operand tables are rebuilt)."""
    dims = (4, 6, 4, 8)
    ph = random_phases(620)
    u, lat = lattice(dims, 621, ph)
    w1, w2 = synth.ptc_weights(8, seed=622)
    w1 = w1 + random_weights(8, 1, 623, 0.05)
    net = W.wl_ptc_create(w1, w2)
    r = f32(synth.gaussian_spinor(dims, seed=624))
    e = f32(synth.gaussian_spinor(dims, seed=625))
    out = lat.new(W.WL_FULL, W.WL_F32)
    rin = lat.pack(r, W.WL_FULL, W.WL_F32)
    W.wl_ptc_apply(lat.ctx, net, out, rin)
    W.wl_ptc_accumulate(lat.ctx, net, rin, lat.pack(e, W.WL_FULL, W.WL_F32), 1.0)
    W.wl_ptc_step(net, 1e-2)
    n1, n2 = W.wl_ptc_get_weights(net, 8)
    W.wl_ptc_apply(lat.ctx, net, out, rin)
    want, _ = ptc.net_apply(r, bf16_round(n1), bf16_round(n2), u, ph)
    assert rel(lat.unpack(out, W.WL_FULL, W.WL_F32).reshape(want.shape), want) < TOL32
    W.wl_ptc_destroy(net)


@pytest.mark.parametrize("channels,dims", [(8, (2, 2, 2, 2)), (8, (6, 6, 4, 8)), (5, (6, 2, 2, 6)), (4, (4, 6, 4, 12)),
                                           (3, (2, 6, 2, 10)), (2, (4, 2, 6, 2)), (1, (4, 2, 6, 2)),
                                           (9, (2, 2, 4, 6))])
def test_gradients_of_padded_and_ragged_networks(channels, dims):
    """Gradients of both losses by the fused backward kernel (2 to 8 channels, padded to 4 or 8) and by the
    layer kernels (1 and 9): fewer points than one tile of 16, partial last tiles, one to five blocks of 16
    tiles.  FP32 sums against the FP64 oracle with the same BF16 weights: 1e-4 normwise, as the other
    gradient tests."""
    ph = random_phases(630 + channels)
    u, lat = lattice(dims, 631, ph)
    w1, w2 = synth.ptc_weights(channels, seed=632)
    w1 = w1 + random_weights(channels, 1, 633, 0.05)
    w2 = w2 + random_weights(1, channels, 634, 0.05)
    w1b, w2b = bf16_round(w1), bf16_round(w2)
    net = W.wl_ptc_create(w1, w2)
    r, e = (f32(synth.gaussian_spinor(dims, seed=635 + k)) for k in range(2))
    rin, ein = (lat.pack(f, W.WL_FULL, W.WL_F32) for f in (r, e))
    W.wl_ptc_accumulate(lat.ctx, net, rin, ein, 0.5)
    W.wl_ptc_accumulate_residual(lat.ctx, net, rin, 0.12, 0.5)
    g1, g2 = W.wl_ptc_get_grads(net, channels)
    loss = W.wl_ptc_step(net, 1e-3)
    la, a1, a2 = ptc.loss_and_grads([(r, e)], w1b, w2b, u, ph)
    lb, b1, b2 = ptc.loss_and_grads_residual([r], w1b, w2b, u, ph, 0.12)
    for got, want in ((g1, 0.5 * (a1 + b1)), (g2, 0.5 * (a2 + b2))):
        assert rel(got, want) < 1e-4
        for p in range(9):
            assert rel(got[p], want[p]) < 1e-3, p
    assert abs(loss - 0.5 * (la + lb)) < 1e-5 * loss
    W.wl_ptc_destroy(net)


@pytest.mark.parametrize("channels,adjoint", [(8, False), (8, True), (5, False), (4, True)])
def test_network_errors_are_roundings_only(channels, adjoint):
    """The matrix-core network's error holds no error of the map itself.  d = output - oracle, projected on every
    path's transported input t_q: E_q = sum_x d t_q^+ / (sum |t_q|^2 / 4).  Roundings that differ from site to site
    leave |E_q[s, t]|^2 ~ (|d| / |t_q|)^2 / (3 V) per entry, so sqrt(sum over 9 x 16 entries) is about
    12 (|d| / |t|) / sqrt(3 V), to a few per cent (288 independent numbers); twice that is allowed.  (Products
    cut off next to a weight of order one gave three to six times it.)"""
    dims = (12, 10, 14, 22)
    ph = random_phases(660 + channels)
    u, lat = lattice(dims, 661, ph)
    w1, w2 = synth.ptc_weights(channels, seed=662)
    net = W.wl_ptc_create(w1, w2)
    w1b, w2b = bf16_round(w1), bf16_round(w2)
    f = f32(synth.gaussian_spinor(dims, seed=663))
    out = lat.new(W.WL_FULL, W.WL_F32)
    W.wl_ptc_apply(lat.ctx, net, out, lat.pack(f, W.WL_FULL, W.WL_F32), adjoint=adjoint)
    if adjoint:
        want = ptc.layer_adjoint(ptc.layer_adjoint([f], w2b, u, ph), w1b, u, ph)[0]
    else:
        want, _ = ptc.net_apply(f, w1b, w2b, u, ph)
    d = lat.unpack(out, W.WL_FULL, W.WL_F32).reshape(want.shape) - want
    n2, total = float(np.linalg.norm(f.ravel())) ** 2, 0.0
    for p in range(ptc.NPATH):
        t = ptc.transport(f, u, ph, p)
        e = np.tensordot(d, t.conj(), axes=([0, 1, 2, 3, 5], [0, 1, 2, 3, 5])) / (n2 / 4)
        total += float(np.linalg.norm(e)) ** 2
    noise = 12 * float(np.linalg.norm(d.ravel())) / np.sqrt(n2) / np.sqrt(3 * np.prod(dims))
    print("map error %.2e, of roundings alone %.2e" % (np.sqrt(total), noise))
    assert np.sqrt(total) <= 2 * noise
    W.wl_ptc_destroy(net)


@pytest.mark.parametrize("channels,adjoint", [(8, False), (4, True), (6, False)])
def test_network_of_numbers_near_the_largest(channels, adjoint):
    """Inputs up to the largest FP32 number (above 3.3961e38 a BF16 rounding is infinite), with weights small
    enough for finite outputs: the network and its adjoint against the oracle, at the FP32 tolerance."""
    dims = (4, 4, 6, 4)
    ph = random_phases(670 + channels)
    u, lat = lattice(dims, 671, ph)
    w1, w2 = synth.ptc_weights(channels, seed=672)
    w1, w2 = 0.25 * w1, 0.5 * w2
    net = W.wl_ptc_create(w1, w2)
    w1b, w2b = bf16_round(w1), bf16_round(w2)
    f = np.zeros(dims[::-1] + (4, 3), dtype=np.complex128)
    big = [float(x) for x in (np.float32(3.4028235e38), np.float32(3.4e38), np.float32(3.3962e38))]
    f[0, 0, 0, 0, 0, 0], f[1, 3, 2, 1, 3, 2], f[3, 1, 0, 2, 1, 1] = big[0], 1j * big[1], -big[2]
    out = lat.new(W.WL_FULL, W.WL_F32)
    W.wl_ptc_apply(lat.ctx, net, out, lat.pack(f, W.WL_FULL, W.WL_F32), adjoint=adjoint)
    if adjoint:
        want = ptc.layer_adjoint(ptc.layer_adjoint([f], w2b, u, ph), w1b, u, ph)[0]
    else:
        want, _ = ptc.net_apply(f, w1b, w2b, u, ph)
    got = lat.unpack(out, W.WL_FULL, W.WL_F32).reshape(want.shape)
    assert np.abs(want).max() < 3e38
    assert np.isfinite(got).all()
    assert rel(got / big[0], want / big[0]) < TOL32
    W.wl_ptc_destroy(net)


@pytest.mark.parametrize("channels,nrhs,adjoint", [(6, 1, False), (3, 2, True), (2, 1, False), (7, 1, True),
                                                   (5, 3, False)])
def test_network_of_tiny_numbers(channels, nrhs, adjoint):
    """Inputs down to the smallest FP32 numbers: the network of 2^-k f is 2^-k times that of f, at the FP32
    tolerance (2^-122: BF16 parts alone hold 11 bits of such a number; 2^-136: FP32 holds 13 itself, so the
    oracle is fed the FP32 numbers and the outputs may be a rounding of 2^-150 per addition off).  One
    right-hand side of zeros among tiny ones stays zero."""
    dims = (6, 4, 2, 6)
    ph = random_phases(680 + channels)
    u, lat = lattice(dims, 681, ph)
    w1, w2 = synth.ptc_weights(channels, seed=682)
    w1 = w1 + random_weights(channels, 1, 683, 0.05)
    w2 = w2 + random_weights(1, channels, 684, 0.05)
    net = W.wl_ptc_create(w1, w2)
    w1b, w2b = bf16_round(w1), bf16_round(w2)

    def apply(fields):
        out = lat.new(W.WL_FULL, W.WL_F32, nrhs)
        stack = np.stack([f.reshape(-1, 4, 3) for f in fields])
        W.wl_ptc_apply(lat.ctx, net, out, lat.pack(stack, W.WL_FULL, W.WL_F32, nrhs), nrhs=nrhs, adjoint=adjoint)
        got = lat.unpack(out, W.WL_FULL, W.WL_F32, nrhs)
        return [(got[r] if nrhs > 1 else got).reshape(fields[0].shape) for r in range(nrhs)]

    def oracle(f):
        if adjoint:
            return ptc.layer_adjoint(ptc.layer_adjoint([f], w2b, u, ph), w1b, u, ph)[0]
        return ptc.net_apply(f, w1b, w2b, u, ph)[0]

    base = [f32(synth.gaussian_spinor(dims, seed=685 + r)) for r in range(nrhs)]
    base[-1] = base[-1] * (nrhs == 1)
    for k, tol in ((100, TOL32), (112, TOL32), (122, TOL32), (136, 100 * 2.0 ** -14)):
        fields = [f32(f * 2.0 ** -k) for f in base]
        for f, got in zip(fields, apply(fields)):
            want = oracle(f)
            if np.any(f):
                print(k, rel(got * 2.0 ** k, want * 2.0 ** k))
                assert rel(got * 2.0 ** k, want * 2.0 ** k) < tol, k
            else:
                assert not np.any(got)
    W.wl_ptc_destroy(net)


@pytest.mark.parametrize("channels,nrhs,adjoint", [(1, 2, False), (1, 3, True), (9, 2, True), (9, 3, False)])
def test_networks_on_the_layer_kernels(channels, nrhs, adjoint):
    """Networks of one or more than eight channels take the layer kernels (two to eight the matrix cores, padded to
    four or eight): M (M^+) of several right-hand sides against the oracle's two layers.  8x6x10x12 x nrhs leaves the gather's last blocks partly empty and their
    number no multiple of the eight XCDs."""
    dims = (8, 6, 10, 12)
    ph = random_phases(690 + channels)
    u, lat = lattice(dims, 691, ph)
    w1, w2 = synth.ptc_weights(channels, seed=692)
    w1 = w1 + random_weights(channels, 1, 693, 0.05)
    w2 = w2 + random_weights(1, channels, 694, 0.05)
    w1b, w2b = bf16_round(w1), bf16_round(w2)
    net = W.wl_ptc_create(w1, w2)
    fields = [f32(synth.gaussian_spinor(dims, seed=695 + r)) for r in range(nrhs)]
    stack = np.stack([f.reshape(-1, 4, 3) for f in fields])
    out = lat.new(W.WL_FULL, W.WL_F32, nrhs)
    W.wl_ptc_apply(lat.ctx, net, out, lat.pack(stack, W.WL_FULL, W.WL_F32, nrhs), nrhs=nrhs, adjoint=adjoint)
    got = lat.unpack(out, W.WL_FULL, W.WL_F32, nrhs)
    for r, f in enumerate(fields):
        if adjoint:
            want = ptc.layer_adjoint(ptc.layer_adjoint([f], w2b, u, ph), w1b, u, ph)[0]
        else:
            want, _ = ptc.net_apply(f, w1b, w2b, u, ph)
        assert rel(got[r].reshape(want.shape), want) < TOL32, r
    W.wl_ptc_destroy(net)


@pytest.mark.parametrize("channels,dims", [(8, (10, 14, 6, 22)), (3, (10, 14, 6, 22)), (2, (18, 14, 22, 24))])
def test_gradients_where_blocks_take_several_tiles(channels, dims):
    """The fused gradient kernel with more than 512 tiles of 16 points, where a block takes several (the ragged
    lattices of the test above have at most 72, one a block): 10x14x6x22
    has 1,156 tiles, three a block (the last block one, one block across the parities, a partial tile at the end
    of each parity), 18x14x22x24 has 8,316, sixteen a block (the last block twelve).  A tile left out would be
    1e-4 to 1e-3 of the sum; FP32 arithmetic with the oracle's BF16 weights: TOL32 normwise."""
    ph = random_phases(700 + channels)
    u, lat = lattice(dims, 701, ph)
    w1, w2 = synth.ptc_weights(channels, seed=702)
    w1 = w1 + random_weights(channels, 1, 703, 0.05)
    w2 = w2 + random_weights(1, channels, 704, 0.05)
    net = W.wl_ptc_create(w1, w2)
    r, e = (f32(synth.gaussian_spinor(dims, seed=705 + k)) for k in range(2))
    W.wl_ptc_accumulate(lat.ctx, net, lat.pack(r, W.WL_FULL, W.WL_F32), lat.pack(e, W.WL_FULL, W.WL_F32), 1.0)
    g1, g2 = W.wl_ptc_get_grads(net, channels)
    loss = W.wl_ptc_step(net, 1e-3)
    want_loss, a1, a2 = ptc.loss_and_grads([(r, e)], bf16_round(w1), bf16_round(w2), u, ph)
    print("gradient errors", rel(g1, a1), rel(g2, a2), "loss", abs(loss - want_loss) / want_loss)
    for got, want in ((g1, a1), (g2, a2)):
        assert rel(got, want) < TOL32
        for p in range(9):
            assert rel(got[p], want[p]) < 1e-4, p
    assert abs(loss - want_loss) < 1e-5 * want_loss
    W.wl_ptc_destroy(net)
