"""GPU parity of the warm start: the BF16 matrix-core surrogate and the
profile loader, through the C ABI, against the FP64 oracle.

Surrogate tolerances.  The oracle's quantised mode rounds weights, layer
inputs and pre-activation gradients to bfloat16 at the same points as the
kernels.  What remains is FP32 accumulation order and FP32 tanh / features,
and those are not small at the output: an FP32 difference of one unit in the
last place flips a bfloat16 rounding with probability |delta| / ulp_bf16, a
flip moves that activation by 2^-8 relative, and every activation feeds
5 x 64 pre-activations of the next layer, so flips cascade.  Emulating the
kernels' arithmetic in numpy float32 against the FP64 oracle gives relative
L2 errors from 1e-7 (no flip) up to 2e-3 on these shapes.  The bars are
therefore:
  * forward outputs: relative L2 <= 1e-2 per sample and max error <= 2e-2 of
    the sample's max (a wrong border tap or a dropped bias exceeds both at
    X = 64);
  * gradients of every layer (weights and biases): relative L2 <= 1e-2;
  * Adam: the closed-form update of the kernel's own gradients to 1e-6 of lr;
  * a short training run: losses within 2 % of the oracle's trajectory.
Profile loader: counts, ids, positions and free-flight counters bit-exact,
velocities to FP32 rounding, deposit and field as in the uniform load.
"""
import math

import numpy as np
import pytest

from gpu_compare import by_id, deposit_matches, field_matches, gpu_state, oracle_from_gpu, restart_step_check
from oracle import surrogate_oracle as SO
from paper_2605_07083_amd import presets

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available(), "GPU tests need a ROCm device"
    return T


@pytest.fixture(scope="module")
def sur(torch):
    from paper_2605_07083_amd import surrogate as S
    S.lib()
    return S


def _say(msg):
    print(msg, flush=True)


def _params(n, seed):
    d = presets.surrogate_params(n, seed)
    return np.stack([d["gamma_emit"], d["T_K"], d["V"], d["ng"]], axis=1)


def _target39(u, k):
    """Smooth targets for all output channels: the three profiles, then
    quantile-like channels increasing with the channel index."""
    rows = [u * (1 + 0.1 * k), np.log(0.2 + u), np.log(1.2 - u)]
    for c in range(3, SO.N_OUT):
        j = (c - 3) % 9
        rows.append(0.3 * (j - 4) + 0.2 * np.sin(3 * u + c + k))
    return np.stack(rows)


def _rel(a, b):
    return float(np.linalg.norm(np.asarray(a, np.float64) - b) / max(np.linalg.norm(b), 1e-300))


@pytest.mark.parametrize("B,X", [(1, 64), (3, 192), (2, 2048), (32, 2048)])
def test_forward_matches_oracle(sur, torch, B, X):
    _say("case: surrogate forward B=%d X=%d" % (B, X))
    W, b = presets.surrogate_test_weights(11)
    p = _params(B, 21)
    net = sur.Surrogate(B, X, device="cuda:0")
    net.set_weights(W, b)
    got = net.forward(p).cpu().numpy()
    p32 = p.astype(np.float32).astype(np.float64)     # the kernel receives FP32 parameters
    ref = SO.forward(W, b, SO.features(p32, X), quantize=True)
    for k in range(B):
        e = _rel(got[k], ref[k])
        m = np.max(np.abs(got[k] - ref[k])) / np.max(np.abs(ref[k]))
        _say("  sample %d rel L2 %.3g, max err / max %.3g" % (k, e, m))
        assert e <= 1e-2 and m <= 2e-2
    # weights round-trip through the packed layout
    W2, b2 = net.weights()
    assert all(np.array_equal(x, y) for x, y in zip(W, W2)) and all(np.array_equal(x, y) for x, y in zip(b, b2))


# X = 256: one whole slice of the backward kernel; 320: a second slice of 64
# positions (a part shorter than the LDS part); 64: one short part with the
# sample's zero padding on both sides; 2048: eight slices per sample
@pytest.mark.parametrize("B,X", [(2, 256), (3, 320), (1, 64), (2, 2048)])
def test_gradients_and_adam_match_oracle(sur, torch, B, X):
    lr = 1e-3
    _say("case: surrogate gradients B=%d X=%d" % (B, X))
    W, b = presets.surrogate_test_weights(12)
    p = _params(B, 22)
    rng = np.random.default_rng(5)
    u = (np.arange(X) + 0.5) / X
    target = np.stack([_target39(u, k) for k in range(B)])
    target = (target + 0.01 * rng.normal(size=target.shape)).astype(np.float32)
    net = sur.Surrogate(B, X, device="cuda:0")
    net.set_weights(W, b)
    loss = net.train_step(p, target, lr)
    gW, gb = net.grads()
    p32 = p.astype(np.float32).astype(np.float64)
    f = SO.features(p32, X)
    lo, oW, ob = SO.loss_and_grads(W, b, f, target.astype(np.float64), quantize=True)
    _say("  loss gpu %.9g oracle %.9g" % (loss, lo))
    assert loss == pytest.approx(lo, rel=1e-4)
    for l in range(6):
        ew, eb = _rel(gW[l], oW[l]), _rel(gb[l], ob[l])
        _say("  layer %d grad rel L2: W %.3g b %.3g" % (l, ew, eb))
        assert ew <= 1e-2 and eb <= 1e-2
    # Adam step 1 from zero moments on the kernel's own gradients:
    # w1 = w0 - lr g / (|g| + eps)
    W1, b1 = net.weights()
    for l in range(6):
        for w0, w1, g in ((W[l], W1[l], gW[l]), (b[l], b1[l], gb[l])):
            exp = w0.astype(np.float64) - lr * g / (np.abs(g.astype(np.float64)) + 1e-8)
            assert np.max(np.abs(w1 - exp)) <= 1e-6 * lr + 1e-7 * np.abs(exp).max()


def test_training_trajectory_matches_oracle(sur, torch):
    B, X, lr, steps = 2, 128, 2e-3, 12
    _say("case: surrogate training trajectory, %d steps" % steps)
    W, b = presets.surrogate_test_weights(13)
    p = _params(B, 23)
    u = (np.arange(X) + 0.5) / X
    target = np.stack([_target39(u, 0) for _ in range(B)]).astype(np.float32)
    net = sur.Surrogate(B, X, device="cuda:0")
    net.set_weights(W, b)
    f = SO.features(p.astype(np.float32).astype(np.float64), X)
    oW = [w.astype(np.float64) for w in W]
    ob = [v.astype(np.float64) for v in b]
    mW = [np.zeros_like(w) for w in oW]; vW = [np.zeros_like(w) for w in oW]
    mb = [np.zeros_like(v) for v in ob]; vb = [np.zeros_like(v) for v in ob]
    lg, lo = [], []
    for t in range(1, steps + 1):
        lg.append(net.train_step(p, target, lr))
        r = SO.train_step(oW, ob, mW, vW, mb, vb, t, f, target.astype(np.float64), lr)
        lo.append(r[0])
        oW, ob, mW, vW, mb, vb = r[3], r[4], r[5], r[6], r[7], r[8]
    _say("  gpu    %s" % np.array2string(np.array(lg), precision=5))
    _say("  oracle %s" % np.array2string(np.array(lo), precision=5))
    assert np.allclose(lg, lo, rtol=2e-2)
    assert lg[-1] < 0.8 * lg[0]


def test_densities_are_exp_of_forward(sur, torch):
    B, X = 3, 128
    W, b = presets.surrogate_test_weights(14, scale=0.5)
    p = _params(B, 24)
    net = sur.Surrogate(B, X, device="cuda:0")
    net.set_weights(W, b)
    out = net.forward(p).cpu().numpy().astype(np.float64)
    n0 = np.array([1e16, 2e16, 5e15])
    d = net.densities(p, n0).cpu().numpy()
    assert np.allclose(d[:, 0, :], n0[:, None] * np.exp(out[:, 1, :]), rtol=1e-12)
    assert np.allclose(d[:, 1, :], n0[:, None] * np.exp(out[:, 2, :]), rtol=1e-12)
    # the loader's state: densities, V phi/V, quantile channels times the 1 eV speeds
    st = net.state(p, n0).cpu().numpy()
    q_e, m_e, m_i = 1.602176634e-19, 9.1093837015e-31, 6.6464731e-27 - 9.1093837015e-31
    V = p[:, 2].astype(np.float32).astype(np.float64)
    assert np.allclose(st[:, 0:2, :], d, rtol=1e-12)
    assert np.allclose(st[:, 2, :], V[:, None] * out[:, 0, :], rtol=1e-12)
    assert np.allclose(st[:, 3:21, :], out[:, 3:21, :] * np.sqrt(q_e / m_e), rtol=1e-12)
    assert np.allclose(st[:, 21:39, :], out[:, 21:39, :] * np.sqrt(q_e / m_i), rtol=1e-12)


def test_surrogate_rejects_bad_shapes(sur, torch):
    net = sur.Surrogate(2, 64, device="cuda:0")
    with pytest.raises(ValueError):
        net.forward(_params(3, 1))
    from paper_2605_07083_amd import pic
    with pytest.raises(pic.PicError) as e:
        sur.Surrogate(2, 100, device="cuda:0")
    assert e.value.code == pic.PIC_EINVAL


# ---------------------------------------------------------------------------
# warm-start loader
# ---------------------------------------------------------------------------
def _profiles(cfg, seed, scale=1.0):
    """A sheath-like synthetic profile pair with fractional counts per cell."""
    rng = np.random.default_rng(seed)
    N = cfg["N"]
    u = (np.arange(N) + 0.5) / N
    ne = cfg["n0"] * scale * (0.15 + 0.85 * np.sin(np.pi * u) ** 0.5) * (1 + 0.05 * rng.normal(size=N))
    ni = cfg["n0"] * scale * (0.4 + 0.6 * np.sin(np.pi * u) ** 0.3) * (1 + 0.05 * rng.normal(size=N))
    return ne, ni


def _check_load(O, cfg, h, ne, ni, d=0):
    st, t = gpu_state(h, d)
    s = O.Sim(cfg)
    s.load_profiles(ne, ni)
    for sp in (0, 2):
        g, o = by_id(st[sp]), by_id(s.particles(sp))
        assert np.array_equal(g["id"], o["id"])
        assert np.array_equal(g["z"], o["z"])
        assert np.array_equal(g["tc"], o["tc"])
        for c in ("vx", "vy", "vz"):
            assert np.max(np.abs(g[c] - o[c].astype(np.float32)) / np.abs(o[c]).max()) < 1e-6
    assert len(st[1]["id"]) == 0
    assert t["next_id"] == s.next_id
    assert list(t["n_live"]) == [s.count(0), 0, s.count(2)]
    assert deposit_matches(O, cfg, h, st, d) == []
    s2 = oracle_from_gpu(O, cfg, st, t)
    assert field_matches(O, cfg, h, s2, d) == []


def test_profile_load_matches_oracle(torch, O):
    from paper_2605_07083_amd import pic
    cfg = presets.scaled(presets.tiny(), gamma_emit=1e21)
    ne, ni = _profiles(cfg, 1)
    _say("case: profile load, tiny diode")
    dens = torch.tensor(np.stack([ne, ni])[None], dtype=torch.float64, device="cuda:0")
    h = pic.Handle(cfg, densities=dens)
    _check_load(O, cfg, h, ne, ni)
    _say("case: restart parity from the profile load, 30 steps")
    assert restart_step_check(O, cfg, h, 30) == []


def test_profile_load_batched(torch, O):
    from paper_2605_07083_amd import pic
    cfgs = [presets.scaled(presets.tiny(), diode=d, gamma_emit=1e21) for d in range(3)]
    cfgs[1]["N"] = 128
    prof = [_profiles(c, 10 + d, scale=0.5 + 0.3 * d) for d, c in enumerate(cfgs)]
    nmax = 256
    arr = np.zeros((3, 2, nmax))
    for d, (ne, ni) in enumerate(prof):
        arr[d, 0, :len(ne)] = ne
        arr[d, 1, :len(ni)] = ni
    _say("case: profile load, 3 diodes (N 256/128/256)")
    h = pic.Handle(cfgs, densities=torch.tensor(arr, device="cuda:0"))
    for d in range(3):
        _check_load(O, cfgs[d], h, *prof[d], d=d)


@pytest.mark.parametrize("cells,per_cell,electrons",
                         [(2, 500, 1.0), (3, 40, 0.0), (5, 40, 0.5), (256, 100, 0.0), (1025, 20, 0.9), (2047, 200, 1.0),
                          (2048, 60, 0.0), (2048, 300, 0.0), (2047, 400, 0.1)])
def test_field_of_balanced_and_bare_charge(torch, O, cells, per_cell, electrons):
    """The exact potential on grids around the scans' four nodes per thread,
    with charge that 64-bit sums hold and, bare ions of the last two cases
    (sum of |R| times N above 2^61), charge that needs the 128-bit ones."""
    from paper_2605_07083_amd import pic
    cfg = presets.scaled(presets.tiny(), N=cells, n_load=cells * per_cell, gamma_emit=1e21)
    ne, ni = _profiles(cfg, 5)
    ne = ne * electrons
    _say("case: field of %d cells, %d per cell, electrons %.1f" % (cells, per_cell, electrons))
    h = pic.Handle(cfg, densities=torch.tensor(np.stack([ne, ni])[None], dtype=torch.float64, device="cuda:0"))
    st, t = gpu_state(h, 0)
    assert deposit_matches(O, cfg, h, st, 0) == []
    assert field_matches(O, cfg, h, oracle_from_gpu(O, cfg, st, t), 0) == []
    assert restart_step_check(O, cfg, h, 2) == []
    H = [h.hist(0, s) for s in range(3)]
    wide = float(np.abs((H[2] - H[0] - H[1])[1:-1].astype(float)).sum()) * cells > 2.0 ** 61
    assert wide == (per_cell >= 300 and electrons < 0.5)
    h.close()


def test_profile_load_errors(torch):
    from paper_2605_07083_amd import pic
    cfg = presets.tiny()
    N = cfg["N"]
    bad = np.ones((1, 2, N)) * cfg["n0"]
    bad[0, 1, 7] = -1.0
    with pytest.raises(pic.PicError) as e:
        pic.Handle(cfg, densities=torch.tensor(bad, device="cuda:0"))
    assert e.value.code == pic.PIC_ENAN
    big = np.ones((1, 2, N)) * cfg["n0"] * 3.0
    with pytest.raises(pic.PicError) as e:
        pic.Handle(cfg, densities=torch.tensor(big, device="cuda:0"))
    assert e.value.code == pic.PIC_ENOSPACE
    zero = np.zeros((1, 2, N))
    h = pic.Handle(cfg, densities=torch.tensor(zero, device="cuda:0"))
    t = h.tally(0)
    assert list(t["n_live"]) == [0, 0, 0]
    h.step(5)
    h.sync()
    with pytest.raises(ValueError):
        pic.Handle(cfg, densities=torch.zeros((1, 2, N + 1), dtype=torch.float64, device="cuda:0"))


# ---------------------------------------------------------------------------
# warm-start state loader (densities, potential, velocity quantiles)
# ---------------------------------------------------------------------------
def _state(cfg, seed, scale=1.0):
    """Densities as _profiles, a sheath-like potential and per-cell quantile
    vectors of a skewed, drifting distribution (unsorted in some cells), with
    a few cells above the energy limit so the clamp is exercised."""
    from paper_2605_07083_amd import pic
    rng = np.random.default_rng(seed + 100)
    N = cfg["N"]
    ne, ni = _profiles(cfg, seed, scale)
    u = (np.arange(N) + 0.5) / N
    L = np.array(pic.STATE_LEVELS)
    st = np.zeros((pic.STATE_ROWS, N))
    st[0], st[1] = ne, ni
    st[2] = cfg["V"] * u ** 0.7
    for q, (vth, drift) in enumerate(((6e5, 2e5), (2.5e3, -8e3))):
        base_z = drift * (1 - u)[None, :] + vth * (L[:, None] - 0.5) * (1 + 0.3 * rng.random((9, N)))
        base_p = vth * (0.2 + L[:, None]) * (1 + 0.2 * rng.random((9, N)))
        base_z[:, ::17] = base_z[::-1, ::17]           # unordered quantiles in some cells
        base_z[8, ::31] *= 40.0                         # some far above the energy limit
        st[3 + 18 * q:12 + 18 * q] = base_z
        st[12 + 18 * q:21 + 18 * q] = base_p
    return st


def test_state_load_matches_oracle(torch, O):
    from paper_2605_07083_amd import pic
    cfg = presets.scaled(presets.tiny(), gamma_emit=1e21)
    st = _state(cfg, 3)
    _say("case: state load, tiny diode")
    h = pic.Handle(cfg, state=torch.tensor(st[None], dtype=torch.float64, device="cuda:0"))
    g, t = gpu_state(h, 0)
    s = O.Sim(cfg)
    s.load_state(st)
    for sp in (0, 2):
        a, o = by_id(g[sp]), by_id(s.particles(sp))
        assert np.array_equal(a["id"], o["id"])
        assert np.array_equal(a["z"], o["z"])
        assert np.array_equal(a["tc"], o["tc"])
        for c in ("vx", "vy", "vz"):
            assert np.max(np.abs(a[c] - o[c].astype(np.float32)) / np.abs(o[c]).max()) < 1e-6, (sp, c)
    assert t["next_id"] == s.next_id
    assert deposit_matches(O, cfg, h, g, 0) == []
    assert field_matches(O, cfg, h, oracle_from_gpu(O, cfg, g, t), 0) == []
    _say("case: restart parity from the state load, 20 steps")
    assert restart_step_check(O, cfg, h, 20) == []


def test_state_load_batched_and_errors(torch, O):
    from paper_2605_07083_amd import pic
    cfgs = [presets.scaled(presets.tiny(), diode=d, gamma_emit=1e21) for d in range(2)]
    cfgs[1]["N"] = 128
    nmax = 256
    arr = np.zeros((2, pic.STATE_ROWS, nmax))
    sts = [_state(c, 20 + d, 0.7 + 0.3 * d) for d, c in enumerate(cfgs)]
    for d, st in enumerate(sts):
        arr[d, :, :st.shape[1]] = st
    _say("case: state load, 2 diodes (N 256/128)")
    h = pic.Handle(cfgs, state=torch.tensor(arr, device="cuda:0"))
    for d in range(2):
        g, t = gpu_state(h, d)
        s = O.Sim(cfgs[d])
        s.load_state(sts[d])
        for sp in (0, 2):
            a, o = by_id(g[sp]), by_id(s.particles(sp))
            assert np.array_equal(a["z"], o["z"]) and np.array_equal(a["id"], o["id"])
            assert np.max(np.abs(a["vz"] - o["vz"].astype(np.float32)) / np.abs(o["vz"]).max()) < 1e-6
    bad = arr[:1].copy()
    bad[0, 25, 7] = np.nan
    with pytest.raises(pic.PicError) as e:
        pic.Handle(cfgs[0], state=torch.tensor(bad, device="cuda:0"))
    assert e.value.code == pic.PIC_ENAN
    with pytest.raises(ValueError):
        pic.Handle(cfgs[0], state=torch.zeros((1, 3, 256), dtype=torch.float64, device="cuda:0"))


@pytest.mark.parametrize("cells,per_cell", [(2, 40), (7, 900), (8, 200), (9, 3), (101, 1), (257, 40)])
def test_state_load_over_the_blocks_of_cells(torch, O, cells, per_cell):
    """The loader deals eight cells at a time: grids around that, cells without
    particles and cells of several rounds, against the oracle; the loaded
    stores count as sorted, and steps and re-sorts go on from them."""
    from paper_2605_07083_amd import pic
    cfg = presets.scaled(presets.tiny(), gamma_emit=1e21, N=cells, n_load=cells * per_cell, capacity_factor=3.0)
    st = _state(cfg, 40 + cells)
    st[:2, 3:5] = 0.0
    h = pic.Handle(cfg, state=torch.tensor(st[None], dtype=torch.float64, device="cuda:0"))
    g, t = gpu_state(h, 0)
    s = O.Sim(cfg)
    s.load_state(st)
    for sp in (0, 2):
        a, o = by_id(g[sp]), by_id(s.particles(sp))
        assert np.array_equal(a["id"], o["id"]) and np.array_equal(a["z"], o["z"])
        assert np.array_equal(a["tc"], o["tc"])
        for c in ("vx", "vy", "vz"):
            assert np.max(np.abs(a[c] - o[c].astype(np.float32)) / np.abs(o[c]).max()) < 1e-6, (sp, c)
    assert h.tally(0)["resorts"] == 1
    assert deposit_matches(O, cfg, h, g, 0) == []
    assert restart_step_check(O, cfg, h, 70) == []
    h.close()


@pytest.mark.parametrize("B,X", [(1, 64), (2, 128), (9, 320), (20, 704), (70, 64), (5, 4096), (33, 1216), (64, 2048), (32, 2048), (48, 2048)])
def test_forward_is_the_same_on_every_tiling(sur, torch, B, X):
    """Rows per block follow the batch and the length (32 to 192, the last tile
    ragged); the values do not: a batch equals its samples one at a time, bit
    for bit, and the densities and the state equal the network's channels
    converted in float64 (exp within two units in the last place)."""
    _say("case: forward tilings B=%d X=%d" % (B, X))
    W, b = presets.surrogate_test_weights(23)
    net = sur.Surrogate(B, X, device="cuda:0")
    net.set_weights(W, b)
    p = torch.tensor(_params(B, 31), dtype=torch.float32, device="cuda:0")
    n0 = torch.linspace(1e15, 3e16, B, dtype=torch.float64, device="cuda:0")
    out, dens, state = net.forward(p), net.densities(p, n0), net.state(p, n0)
    for k in sorted({0, B // 2, B - 1}):
        assert torch.equal(net.forward(p[k:k + 1])[0], out[k])
        assert torch.equal(net.state(p[k:k + 1], n0[k:k + 1])[0], state[k])
    assert torch.equal(dens, state[:, :2])
    o = out.cpu().numpy().astype(np.float64)
    v1 = [math.sqrt(1.602176634e-19 / m) for m in (9.1093837015e-31, 6.6464731e-27 - 9.1093837015e-31)]
    ref = np.concatenate([n0.cpu().numpy()[:, None, None] * np.exp(o[:, 1:3]),
                          p[:, 2].double().cpu().numpy()[:, None, None] * o[:, 0:1], o[:, 3:21] * v1[0],
                          o[:, 21:39] * v1[1]], 1)
    assert np.allclose(state.cpu().numpy(), ref, rtol=1e-15 * 4, atol=0.0)


def test_forward_into_an_odd_offset(sur, torch):
    """The caller's output needs no more than a float's alignment."""
    _say("case: forward into an output at an odd element offset")
    W, b = presets.surrogate_test_weights(23)
    B, X = 3, 192
    net = sur.Surrogate(B, X, device="cuda:0")
    net.set_weights(W, b)
    p = _params(B, 31)
    ref = net.forward(p)
    flat = torch.full((B * SO.N_OUT * X + 3,), float("nan"), dtype=torch.float32, device="cuda:0")
    out = flat[1:1 + B * SO.N_OUT * X].view(B, SO.N_OUT, X)
    assert torch.equal(net.forward(p, out), ref)
    assert torch.isnan(flat[:1]).all() and torch.isnan(flat[1 + B * SO.N_OUT * X:]).all()


@pytest.mark.parametrize("B,X", [(2, 64), (4, 320), (8, 704), (16, 64), (32, 1216), (4, 4096)])
def test_train_step_on_every_tiling(sur, torch, B, X):
    """The training step's rows per block follow the batch and the length.  Its
    loss is the mean of the samples' own and its gradients the mean of theirs:
    with a power of two samples the gradients at the output scale exactly, so
    only FP32 sums of at most a few hundred partials differ (6e-8 times the
    root of their number, below 1e-5)."""
    _say("case: train step tilings B=%d X=%d" % (B, X))
    W, b = presets.surrogate_test_weights(29)
    p = torch.tensor(_params(B, 37), dtype=torch.float32, device="cuda:0")
    u = np.linspace(0.5 / X, 1 - 0.5 / X, X)
    t = torch.tensor(np.stack([_target39(u, k) for k in range(B)]), dtype=torch.float32, device="cuda:0")
    net = sur.Surrogate(B, X, device="cuda:0")
    net.set_weights(W, b)
    loss = net.train_step(p, t, 1e-3)
    gw, gb = net.grads()
    losses, sw, sb = [], [np.zeros_like(x, np.float64) for x in gw], [np.zeros_like(x, np.float64) for x in gb]
    for k in range(B):
        net.set_weights(W, b)
        losses.append(net.train_step(p[k:k + 1], t[k:k + 1], 1e-3))
        for s, g in zip(sw + sb, sum(net.grads(), [])):
            s += g.astype(np.float64) / B
    assert abs(loss - np.mean(losses)) <= 1e-12 * loss
    for s, g in zip(sw + sb, gw + gb):
        assert _rel(g, s) <= 1e-5


@pytest.mark.parametrize("B,X", [(1, 64), (6, 64), (3, 128), (5, 320), (2, 576), (3, 1024)])
def test_training_within_its_workspace(sur, torch, B, X):
    """Samples of 64, 128 and 320 positions sum their gradients in several
    launches, others in one.  Either way a step writes nothing beyond its
    workspace, and a batch below the handle's largest gives the same loss,
    weights and gradients, bit for bit, as a handle of exactly that batch."""
    import ctypes as C
    _say("case: training workspace B=%d X=%d" % (B, X))
    W, b = presets.surrogate_test_weights(41)
    p = torch.tensor(_params(B, 43), dtype=torch.float32, device="cuda:0")
    u = np.linspace(0.5 / X, 1 - 0.5 / X, X)
    t = torch.tensor(np.stack([_target39(u, k) for k in range(B)]), dtype=torch.float32, device="cuda:0")
    got = []
    for most in (B, B + 3):
        n = sur.workspace_size(most, X)
        net = sur.Surrogate(1, 64, device="cuda:0")
        net.close()
        net.ws = torch.full((n + 65536,), 0xA5, dtype=torch.uint8, device="cuda:0")
        net.max_batch, net.cells, net.h = most, X, C.c_void_p()
        assert sur.lib().sur_create(most, X, C.c_void_p(net.ws.data_ptr()), n,
                                    C.c_void_p(net.stream.cuda_stream), 0, C.byref(net.h)) == 0
        net.set_weights(W, b)
        losses = [net.train_step(p, t, 1e-3) for _ in range(3)]
        got.append((losses, [x for v in net.weights() + net.grads() for x in v]))
        assert bool((net.ws[n:] == 0xA5).all())
        net.close()
    assert got[0][0] == got[1][0]
    assert all(np.array_equal(x, y) for x, y in zip(got[0][1], got[1][1]))


@pytest.mark.parametrize("cells,electrons,ions", [(2049, 1.0, 0.0), (2560, 0.0, 1.0), (4607, 0.9, 1.0),
                                                  (19456, 1.0, 0.1), (32767, 0.0, 1.0), (32767, 1.0, 0.0)])
def test_field_of_tiled_grids(torch, O, cells, electrons, ions):
    """The tiles' aggregates on grids from five tiles to sixty-four, of bare
    charge of either sign (every word of a negative sum has its high bits set)
    and of near balance, over a few launches, against the exact rational solve
    (an FP64 sweep is off by more than the tolerance on the largest grids)."""
    from paper_2605_07083_amd import pic
    cfg = presets.scaled(presets.tiny(), N=cells, n_load=cells * 30, gamma_emit=1e21)
    ne, ni = _profiles(cfg, 5)
    dens = np.stack([ne * electrons, ni * ions])[None]
    _say("case: field of %d cells, electrons %.1f, ions %.1f" % (cells, electrons, ions))
    h = pic.Handle(cfg, densities=torch.tensor(dens, dtype=torch.float64, device="cuda:0"))
    for steps in (0, 1, 3):
        h.step(steps)
        st, t = gpu_state(h, 0)
        assert deposit_matches(O, cfg, h, st, 0) == []
        h.refield()
        assert field_matches(O, cfg, h, oracle_from_gpu(O, cfg, st, t), 0, exact=True) == []
    assert restart_step_check(O, cfg, h, 2, exact_field=True) == []
    h.close()


@pytest.mark.parametrize("cells,per_cell,diodes", [(2, 20000, 1), (8, 6000, 1), (17, 4000, 1), (5, 3000, 3), (130, 700, 1)])
def test_state_load_of_few_cells_with_many_particles(torch, O, cells, per_cell, diodes):
    """Where the cells are too few to fill the chip, several blocks share a
    group's particles: every one is loaded once, as by the oracle."""
    from paper_2605_07083_amd import pic
    _say("case: state load, %d diodes of %d cells x %d" % (diodes, cells, per_cell))
    cfgs = [presets.scaled(presets.tiny(), gamma_emit=1e21, N=cells, n_load=cells * per_cell // (d + 1), diode=d,
                           capacity_factor=3.0) for d in range(diodes)]
    sts = np.stack([_state(c, 60 + d) for d, c in enumerate(cfgs)])
    h = pic.Handle(cfgs, state=torch.tensor(sts, dtype=torch.float64, device="cuda:0"))
    for d, cfg in enumerate(cfgs):
        g, t = gpu_state(h, d)
        s = O.Sim(cfg)
        s.load_state(sts[d])
        for sp in (0, 2):
            a, o = by_id(g[sp]), by_id(s.particles(sp))
            assert np.array_equal(a["id"], o["id"]) and np.array_equal(a["z"], o["z"])
            assert np.array_equal(a["tc"], o["tc"])
            for c in ("vx", "vy", "vz"):
                assert np.max(np.abs(a[c] - o[c].astype(np.float32)) / np.abs(o[c]).max()) < 1e-6
        assert deposit_matches(O, cfg, h, g, d) == []
    h.close()
