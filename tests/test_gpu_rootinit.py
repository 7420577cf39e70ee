"""GPU parity of the learned root initialiser and the guided root finding
against the FP64 oracle, through the C ABI."""
import numpy as np
import pytest
import torch

from paper_2212_10550_amd import synth
from tests import indep
from tests.gpu_util import assert_mixed, dev, host, soa, up

pytestmark = pytest.mark.gpu


def _K():
    from paper_2212_10550_amd import lib as K
    return K


def _params():
    p = synth.make_rootinit_params(seed=4).astype(np.float32)
    p[-27:-3] += np.linspace(0, 0.5, 24, dtype=np.float32)
    return p


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_rootinit_fwd(orc, dtype):
    K = _K()
    w = synth.train_step()
    skel = synth.make_skeleton(0)
    S = 3000
    xp = synth.sample_posed_points(skel, w.B.astype(np.float64), S, 3)
    params = _params()
    bone = torch.empty(S, dtype=torch.int16, device=dev())
    x0 = torch.empty(3, S + 7, device=dev())
    K.rootinit_fwd(soa(xp, S + 7), S, S + 7, up(w.pose_params.reshape(-1)), up(params), up(w.B),
                   K.F32 if dtype == "f32" else K.BF16, bone, x0)
    torch.cuda.synchronize()
    rb, rx0 = orc.rootinit_fwd(xp, w.pose_params, params, w.B)
    gb = host(bone).astype(int)
    agree = gb == rb
    gx = host(x0[:, :S]).T
    print(f"rootinit {dtype}: bone agreement {agree.mean():.4f}, x0 max err {np.abs(gx - rx0)[agree].max():.2e}")
    if dtype == "f32":
        assert agree.mean() > 0.999
        assert_mixed(gx[agree], rx0[agree], 1e-5, "x0")
    else:
        assert agree.mean() > 0.95
        assert np.abs(gx - rx0)[agree].mean() < 1e-2


@pytest.mark.parametrize("nb", [1, 13, 14, 29])
def test_rootinit_bones_and_ragged(orc, nb):
    """Bone counts whose offsets lie in one or both output tiles, up to the
    most; the FP32 form against the oracle (the bars of the test above), and
    the BF16 form on ragged counts bit-equal to the first samples of a longer
    call (samples are independent), writing nothing past the count."""
    K = _K()
    rng = np.random.default_rng(nb)
    w = synth.train_step()
    S = 700
    xp = rng.uniform(0.2, 0.8, (S, 3)).astype(np.float32)
    B = np.ascontiguousarray(np.resize(w.B, (nb, 3, 4))).astype(np.float32)
    pose = rng.normal(0, 0.3, (nb, 6)).astype(np.float32)
    nin, nout = 3 + 6 * nb, nb + 3
    params = np.concatenate([rng.normal(0, 1 / np.sqrt(a), a * b).tolist() + rng.normal(0, 0.1, b).tolist()
                             for a, b in [(nin, 64), (64, 64), (64, nout)]]).astype(np.float32)

    def run(n, dtype, cap=None):
        cap = n if cap is None else cap
        bone = torch.full((S,), -7, dtype=torch.int16, device=dev())
        x0 = torch.full((3, S), -7.0, device=dev())
        Sd = None if cap == n else torch.tensor([n], dtype=torch.int64, device=dev())
        K.rootinit_fwd(soa(xp), cap, S, up(pose.reshape(-1)), up(params), up(B), dtype, bone, x0, S_dev=Sd)
        torch.cuda.synchronize()
        return host(bone).astype(int), host(x0)

    gb, gx = run(S, K.F32)
    rb, rx0 = orc.rootinit_fwd(xp, pose, params, B)
    agree = gb == rb
    assert agree.mean() > 0.99
    assert_mixed(gx.T[agree], rx0[agree], 1e-5, "x0")
    fb, fx = run(S, K.BF16)
    for n, cap in [(1, None), (15, None), (63, None), (64, None), (65, None), (321, None), (130, S), (0, S)]:
        b, x = run(n, K.BF16, cap)
        assert np.array_equal(b[:n], fb[:n]) and np.array_equal(x[:, :n], fx[:, :n]), n
        assert (b[n:] == -7).all() and (x[:, n:] == -7.0).all(), n


def test_rootinit_bf16_steps():
    """BF16 calls and device counts around 32,768 samples, where a wave's step
    goes from 32 samples to 64: each bit-equal to the first samples of the
    longest, nothing written past the count."""
    K = _K()
    w = synth.train_step()
    S = 33000
    xp = soa(synth.sample_posed_points(synth.make_skeleton(0), w.B.astype(np.float64), S, 6).astype(np.float32))
    params, pose, B = up(_params()), up(w.pose_params.reshape(-1)), up(w.B)

    def run(n, cap):
        bone = torch.full((S,), -7, dtype=torch.int16, device=dev())
        x0 = torch.full((3, S), -7.0, device=dev())
        Sd = None if cap == n else torch.tensor([n], dtype=torch.int64, device=dev())
        K.rootinit_fwd(xp, cap, S, pose, params, B, K.BF16, bone, x0, S_dev=Sd)
        return host(bone), host(x0)

    fb, fx = run(S, S)
    for n in (31, 33, 4097, 32767, 32768, 32769, 32801, 32833):
        for cap in (n, S):
            b, x = run(n, cap)
            assert np.array_equal(b[:n], fb[:n]) and np.array_equal(x[:, :n], fx[:, :n]), (n, cap)
            assert (b[n:] == -7).all() and (x[:, n:] == -7.0).all(), (n, cap)


def test_rootinit_bf16_unaligned_params():
    """BF16 initialiser with its parameter block at an address that is not a
    multiple of 16 bytes (the fragments are then gathered one value at a
    time instead of two 16-byte loads): outputs bit-equal to the aligned
    call's."""
    K = _K()
    w = synth.train_step()
    skel = synth.make_skeleton(0)
    S = 2001
    xp = synth.sample_posed_points(skel, w.B.astype(np.float64), S, 5)
    params = _params()
    pa = up(params)
    buf = torch.zeros(params.size + 1, device=dev())
    buf[1:] = pa
    pu = buf[1:]  # 4 bytes past a 16-byte boundary
    assert pu.data_ptr() % 16 != 0
    outs = []
    for p in (pa, pu):
        bone = torch.empty(S, dtype=torch.int16, device=dev())
        x0 = torch.empty(3, S, device=dev())
        K.rootinit_fwd(soa(xp), S, S, up(w.pose_params.reshape(-1)), p, up(w.B), K.BF16, bone, x0)
        torch.cuda.synchronize()
        outs.append((host(bone), host(x0)))
    assert np.array_equal(outs[0][0], outs[1][0])
    assert np.array_equal(outs[0][1].view(np.uint32), outs[1][1].view(np.uint32))


def test_deform_guided(orc):
    K = _K()
    w = synth.train_step()
    skel = synth.make_skeleton(0)
    S = 4000
    xp = synth.sample_posed_points(skel, w.B.astype(np.float64), S, 9)
    ref = orc.deform(xp, w.B, w.W, w.skin_aabb, w.hash_aabb, max_iter=2, details=True)
    rng = np.random.default_rng(6)
    x0 = (ref["xc"] + rng.normal(0, 0.01, ref["xc"].shape)).astype(np.float32)
    x0[::3] = [4.0, -3.0, 5.0]
    guide = rng.integers(0, 24, S).astype(np.int16)
    g = orc.deform_guided(xp, x0, guide, w.B, w.W, w.skin_aabb, w.hash_aabb, max_iter=2)
    Dz, Dy, Dx, nb = w.W.shape
    xc = torch.empty(3, S, device=dev())
    bone = torch.empty(S, dtype=torch.int16, device=dev())
    steps = torch.empty(S, dtype=torch.int16, device=dev())
    nfb = torch.zeros(1, dtype=torch.int32, device=dev())
    ws = torch.empty(K.deform_guided_workspace_size(S, Dx, Dy, Dz), dtype=torch.uint8, device=dev())
    K.snarf_deform_guided(soa(xp), S, S, soa(x0), up(guide), up(w.B), up(w.W), w.skin_aabb, w.hash_aabb, 2, 1e-6,
                          1e-5, xc, bone, None, steps, nfb, ws)
    torch.cuda.synchronize()
    gb = host(bone).astype(int)
    gx = host(xc).T
    gfb = gb != guide  # accepted guided samples keep the guide's bone
    ofb = g["fallback"] == 1
    flips = (gfb != ofb) & ~((gb == guide) & ofb)  # a fallback may pick the guide's bone by chance
    assert flips.mean() < 0.01, flips.mean()
    assert int(nfb.item()) >= ofb.sum() * 0.9
    valid = gb >= 0
    f = indep.lbs_scipy(w.B, w.W, w.skin_aabb)
    assert (np.linalg.norm(f(gx[valid]) - xp[valid], axis=1) < 1e-5).all()
    # every GPU root is one of the distinct roots the full multi-init solve finds
    full = orc.deform(xp, w.B, w.W, w.skin_aabb, w.hash_aabb, details=True)
    both = valid & (full["n_roots"] > 0)
    assert both.mean() > 0.9
    dist = np.linalg.norm(full["roots"][both] - gx[both][:, None, :], axis=2)
    dist = np.where(np.arange(nb)[None, :] < full["n_roots"][both][:, None], dist, np.inf)
    k = dist.argmin(1)
    assert_mixed(gx[both], full["roots"][both][np.arange(both.sum()), k], 1e-5, "guided roots")
    print(f"guided: fallback gpu {int(nfb.item())} oracle {ofb.sum()} of {S}")


@pytest.mark.parametrize("guided", [True, False])
@pytest.mark.parametrize("S,count", [(1, None), (63, None), (65, None), (1000, None), (300, 129), (70, 0)])
def test_deform_order(S, count, guided):
    """Samples in an order where a wave's lie in few cells (they are then
    loaded once and shared) and in one where they do not: the same bits for
    every sample, on ragged counts and under a device count."""
    K = _K()
    w = synth.train_step()
    rng = np.random.default_rng(S)
    skel = synth.make_skeleton(0)
    base = synth.sample_posed_points(skel, w.B.astype(np.float64), max(S // 50, 1), 11)
    xp = (np.repeat(base, 50 + S % 50 + 1, axis=0)[:S] + rng.uniform(-0.004, 0.004, (S, 3))).astype(np.float32)
    x0 = (xp + rng.normal(0, 0.02, (S, 3))).astype(np.float32)
    guide = rng.integers(0, 24, S).astype(np.int16)
    Dz, Dy, Dx, nb = w.W.shape
    n = S if count is None else count

    def run(order):
        xc = torch.full((3, S), -7.0, device=dev())
        bone = torch.full((S,), -7, dtype=torch.int16, device=dev())
        steps = torch.full((S,), -7, dtype=torch.int16, device=dev())
        nfb = torch.zeros(1, dtype=torch.int32, device=dev())
        ws = torch.empty(K.deform_guided_workspace_size(S, Dx, Dy, Dz), dtype=torch.uint8, device=dev())
        Sd = None if count is None else torch.tensor([count], device=dev())
        if guided:
            K.snarf_deform_guided(soa(xp[order]), S, S, soa(x0[order]), up(guide[order]), up(w.B), up(w.W),
                                  w.skin_aabb, w.hash_aabb, 10, 1e-6, 1e-5, xc, bone, None, steps, nfb, ws, S_dev=Sd)
        else:
            K.snarf_deform(soa(xp[order]), S, S, up(w.B), up(w.W), w.skin_aabb, w.hash_aabb, 10, 1e-6, 1e-5, xc, bone,
                           None, steps, ws, S_dev=Sd)
        torch.cuda.synchronize()
        return host(xc), host(bone), host(steps), int(nfb.item())

    order = np.arange(S)
    a = run(order)
    perm = np.concatenate([rng.permutation(n), np.arange(n, S)]).astype(int)
    b = run(perm)
    assert (a[0][:, n:] == -7.0).all() and (a[1][n:] == -7).all()
    assert np.array_equal(a[0][:, perm], b[0]) and np.array_equal(a[1][perm], b[1])
    assert np.array_equal(a[2][perm], b[2]) and a[3] == b[3]


@pytest.mark.parametrize("count", [None, 40, 30000])
def test_guided_either_side_of_the_line(count):
    """65,536 samples and one more: each is the largest or the smallest call
    of a kernel of its own, and a sample's bits are the same in both."""
    K = _K()
    w = synth.train_step()
    rng = np.random.default_rng(5)
    line = 65536
    S = line + 1
    base = synth.sample_posed_points(synth.make_skeleton(0), w.B.astype(np.float64), 4096, 12)
    xp = (np.repeat(base, 17, axis=0)[:S] + rng.uniform(-0.004, 0.004, (S, 3))).astype(np.float32)
    x0 = (xp + rng.normal(0, 0.02, (S, 3))).astype(np.float32)
    guide = rng.integers(0, 24, S).astype(np.int16)
    Dz, Dy, Dx, nb = w.W.shape
    out = []
    for n in (line, S):
        xc = torch.full((3, n), -7.0, device=dev())
        bone = torch.full((n,), -7, dtype=torch.int16, device=dev())
        steps = torch.full((n,), -7, dtype=torch.int16, device=dev())
        nfb = torch.zeros(1, dtype=torch.int32, device=dev())
        ws = torch.empty(K.deform_guided_workspace_size(n, Dx, Dy, Dz), dtype=torch.uint8, device=dev())
        K.snarf_deform_guided(soa(xp[:n]), n, n, soa(x0[:n]), up(guide[:n]), up(w.B), up(w.W), w.skin_aabb,
                              w.hash_aabb, 10, 1e-6, 1e-5, xc, bone, None, steps, nfb, ws,
                              S_dev=None if count is None else torch.tensor([count], device=dev()))
        out.append([host(xc)[:, :line], host(bone)[:line], host(steps)[:line]])
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    assert (out[0][1] >= 0).any()


def test_learned_init_end_to_end():
    """Fit a small initialiser on solver roots of 16 poses, then guided
    solves on held-out poses: every accepted root is a valid root, and most
    samples need no fallback."""
    from paper_2212_10550_amd import rootinit
    data = rootinit.make_dataset(range(1000, 1016), 2048, device="cuda:0")
    params = rootinit.fit(data, epochs=8)
    test = rootinit.make_dataset(range(2000, 2004), 2048, device="cuda:0")
    K = _K()
    w = synth.train_step()
    fallbacks, n = 0, 0
    for p in range(4):
        sel = test["pose_index"] == p
        xp = test["xp"][sel].T.contiguous()
        S = xp.shape[1]
        gd = rootinit.GuidedDeform(params, w, S, device="cuda:0")
        xc = torch.empty(3, S, device=dev())
        bone = torch.empty(S, dtype=torch.int16, device=dev())
        W_t = up(w.W)
        gd.run(xp, S, S, test["pose"][p].contiguous(), test["B"][p].contiguous(), W_t, xc, bone, None, None)
        torch.cuda.synchronize()
        gx = host(xc).T
        B = host(test["B"][p])
        f = indep.lbs_scipy(B, w.W, w.skin_aabb)
        ok = host(bone) >= 0
        assert ok.mean() > 0.99
        assert (np.linalg.norm(f(gx[ok]) - host(xp).T[ok], axis=1) < 1e-5).all()
        fallbacks += int(gd.n_fallback.item())
        n += S
    print(f"learned init: fallback rate {fallbacks / n:.4f}")
    assert fallbacks / n < 0.5
