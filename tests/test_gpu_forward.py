"""GPU parity of the forward stages against the FP64 oracle, through the C ABI.

FP32 path bar: |gpu - oracle| <= 1e-5 * max(1, |oracle|) on points, features,
densities, colours and composited pixels.  Integer work (march) is bit-exact.
"""
import numpy as np
import pytest
import torch

from paper_2212_10550_amd import synth
from tests import indep
from tests.gpu_util import feat_dev, feat_host, assert_mixed, dev, host, soa, up, unpack_bricks

pytestmark = pytest.mark.gpu

TOL = 1e-5


def _K():
    from paper_2212_10550_amd import lib as K
    return K


def _march_gpu(w, cap=None):
    from paper_2212_10550_amd.pipeline import Pipeline
    p = Pipeline(w, cap=cap)
    p.march()
    S = p.read_count()
    torch.cuda.synchronize()
    return p, S


@pytest.mark.parametrize("which", ["tiny", "train_subset", "frame_rows"])
def test_march_bit_exact(orc, which):
    if which == "tiny":
        w = synth.tiny_forward()
    elif which == "train_subset":
        w = synth.train_step()
    else:
        w = synth.full_frame()
        w = synth.ray_subset(w, np.arange(200 * 540, 260 * 540))
    p, S = _march_gpu(w)
    m = orc.march(w.rays_o, w.rays_d, w.occ, w.occ_aabb, w.dt, w.n_per_ray, w.max_steps)
    assert S == m["xs"].shape[0] and S > 0
    np.testing.assert_array_equal(host(p.ray_off), m["ray_off"])
    np.testing.assert_array_equal(host(p.ray_cnt), m["ray_cnt"])
    np.testing.assert_array_equal(host(p.ray_dt), m["ray_dt"])
    np.testing.assert_array_equal(p.soa(p.xs), m["xs"])
    np.testing.assert_array_equal(host(p.ts[:S]), m["ts"])
    np.testing.assert_array_equal(host(p.ray_id[:S]), m["ray_id"])


@pytest.mark.parametrize("G", [16, 37, 128])
def test_occ_pack_brick_layout(G):
    K = _K()
    rng = np.random.default_rng(G)
    occ = (rng.random((G, G, G)) < 0.3).astype(np.uint8)
    bits = torch.full((K.occ_words(G),), -1, dtype=torch.int32, device=dev())
    K.occ_pack(torch.as_tensor(occ, device=dev()), bits)
    full = unpack_bricks(host(bits), G)
    np.testing.assert_array_equal(full[:G, :G, :G], occ.astype(bool))
    assert not full[G:].any() and not full[:, G:].any() and not full[:, :, G:].any()


@pytest.mark.parametrize("box", ["unit", "pow2", "general"])
def test_march_odd_grid_bit_exact(orc, box):
    """A grid size that leaves partial bricks, enough rays for several scan
    chunks (4096 blocks of 4 rays each), and grid boxes whose extents are a
    power of two (cell coordinates by an exact reciprocal) or not (by
    division)."""
    w = synth.full_frame()
    w = synth.ray_subset(w, np.arange(120 * 540, 190 * 540))
    rng = np.random.default_rng(7)
    w.occ = (rng.random((37, 37, 37)) < 0.2).astype(np.uint8)
    if box == "pow2":
        w.occ_aabb = np.array([-0.5, -0.5, -0.5, 1.5, 1.5, 1.5], np.float32)
    elif box == "general":
        w.occ_aabb = np.array([-0.05, -0.02, -0.1, 1.05, 1.0, 1.07], np.float32)
    p, S = _march_gpu(w)
    m = orc.march(w.rays_o, w.rays_d, w.occ, w.occ_aabb, w.dt, w.n_per_ray, w.max_steps)
    assert w.R > 2 * 4 * 4096 and S == m["xs"].shape[0] and S > 0
    np.testing.assert_array_equal(host(p.ray_off), m["ray_off"])
    np.testing.assert_array_equal(host(p.ray_cnt), m["ray_cnt"])
    np.testing.assert_array_equal(p.soa(p.xs), m["xs"])
    np.testing.assert_array_equal(host(p.ray_id[:S]), m["ray_id"])


# ray counts from 32,768 on take one ray per lane: ragged last workgroups,
# step counts that end inside a mask word or span several, every kind of box,
# no grid, a capacity below the count, and (2,100,000 rays) more workgroup
# totals than one scan chunk holds
@pytest.mark.parametrize("R,steps,box,grid,share", [
    (32767, 128, "pow2", 37, 1.0), (32768, 128, "unit", 37, 1.0), (65537, 70, "pow2", 64, 1.0), (70001, 200, "general", 37, 1.0),
    (65791, 1, "unit", 16, 1.0), (66000, 33, "unit", 0, 1.0), (65536, 64, "general", 128, 0.4),
    (2100000, 3, "unit", 16, 1.0)])
def test_march_many_rays_bit_exact(orc, R, steps, box, grid, share):
    from paper_2212_10550_amd import lib as K
    rng = np.random.default_rng(R + steps)
    o = rng.uniform(-0.6, 1.6, (R, 3)).astype(np.float32)
    d = rng.normal(size=(R, 3)).astype(np.float32)
    d[::7, rng.integers(0, 3)] = 0.0  # parallel to two faces
    d[5::9] = np.eye(3, dtype=np.float32)[rng.integers(0, 3, d[5::9].shape[0])]
    aabb = {"unit": [0, 0, 0, 1, 1, 1], "pow2": [-0.5, -0.5, -0.5, 1.5, 1.5, 1.5],
            "general": [-0.05, -0.02, -0.1, 1.05, 1.0, 1.07]}[box]
    aabb = np.array(aabb, np.float32)
    occ = (rng.random((grid,) * 3) < 0.2).astype(np.uint8) if grid else None
    n_per_ray, dt = (steps, 0.0) if not grid else (0, float(np.float32(1.9 / steps)))
    m = orc.march(o, d, occ, aabb, dt, n_per_ray, steps)
    n = m["xs"].shape[0]
    cap = max(1, int(n * share))
    e = lambda *s, dt=torch.float32: torch.full(s, -7, dtype=dt, device=dev())
    bits = None
    if grid:
        bits = torch.empty(K.occ_words(grid), dtype=torch.int32, device=dev())
        K.occ_pack(up(occ), bits)
    xs, ts, rid, off, cnt = e(3, cap), e(cap), e(cap, dt=torch.int32), e(R + 1, dt=torch.int64), e(R, dt=torch.int32)
    rdt, ns, ws = e(R), e(1, dt=torch.int64), e(K.march_workspace_size(R, steps), dt=torch.uint8)
    K.occgrid_march(up(o), up(d), bits, grid, aabb, dt, n_per_ray, steps, xs, ts, rid, cap, off, cnt, rdt, ns, ws)
    torch.cuda.synchronize()
    assert n > 0 and int(ns.item()) == n
    np.testing.assert_array_equal(host(off), m["ray_off"])
    np.testing.assert_array_equal(host(cnt), m["ray_cnt"])
    np.testing.assert_array_equal(host(xs).T, m["xs"][:cap])
    np.testing.assert_array_equal(host(rid), m["ray_id"][:cap])
    np.testing.assert_array_equal(host(ts), m["ts"][:cap])


@pytest.mark.parametrize("R,steps,box,grid", [(20479, 128, "unit", 37), (20480, 128, "unit", 37),
                                              (49151, 1024, "pow2", 64), (49153, 1024, "general", 64),
                                              (65536, 4000, "unit", 0)])
def test_march_line_and_long_rays_bit_exact(orc, R, steps, box, grid):
    """Both sides of the line between the mappings, which rises with the
    steps; and long rays of differing lengths, of which a wave takes the last
    ones one after the other."""
    test_march_many_rays_bit_exact(orc, R, steps, box, grid, 0.05 if steps > 2000 else 1.0)


def test_march_empty_and_capacity(orc):
    w = synth.train_step()
    w0 = synth.ray_subset(w, np.arange(64))
    w0.occ = np.zeros_like(w.occ)
    p, S = _march_gpu(w0)
    assert S == 0 and (host(p.ray_off) == 0).all()
    # too small a buffer: the count is still reported, nothing beyond cap written
    w1 = synth.ray_subset(w, np.arange(0, w.R, 4))
    from paper_2212_10550_amd.pipeline import Pipeline
    p = Pipeline(w1, cap=100)
    p.march()
    torch.cuda.synchronize()
    with pytest.raises(RuntimeError):
        p.read_count()


def _deform_check(orc, w, xp, tag):
    K = _K()
    S = xp.shape[0]
    ld = S + 13  # leading dimension larger than S
    Dz, Dy, Dx, nb = w.W.shape
    xc = torch.zeros(3, ld, device=dev())
    bone = torch.zeros(S, dtype=torch.int16, device=dev())
    resid = torch.zeros(S, device=dev())
    steps = torch.zeros(S, dtype=torch.int16, device=dev())
    ws = torch.empty(K.deform_workspace_size(Dx, Dy, Dz), dtype=torch.uint8, device=dev())
    K.snarf_deform(soa(xp, ld), S, ld, up(w.B), up(w.W), w.skin_aabb, w.hash_aabb, w.max_iter, w.tol_stop,
                   w.tol_valid, xc, bone, resid, steps, ws)
    torch.cuda.synchronize()
    g_x = host(xc[:, :S]).T
    g_b = host(bone).astype(int)
    d = orc.deform(xp, w.B, w.W, w.skin_aabb, w.hash_aabb, w.max_iter, w.tol_stop, w.tol_valid, details=True)
    gv, ov = g_b >= 0, d["bone"] >= 0
    flips = np.nonzero(gv != ov)[0]
    # a validity flip may only happen where the FP64 decision itself is
    # marginal: no init of the oracle converged below the stopping tolerance
    best_r = np.where(np.isfinite(d["init_r"]), d["init_r"], np.inf).min(1)
    assert len(flips) <= max(2, S // 2000), (tag, len(flips))
    assert (best_r[flips] > w.tol_stop).all() if len(flips) else True
    both = gv & ov
    # every GPU root is a valid root: FP64 residual (SciPy interpolant) < tol_valid
    f = indep.lbs_scipy(w.B, w.W, w.skin_aabb)
    r = np.linalg.norm(f(g_x[gv]) - xp[gv], axis=1)
    assert (r < w.tol_valid).all(), (tag, r.max())
    # ... and it matches one of the oracle's distinct valid roots
    dist = np.linalg.norm(d["roots"][both] - g_x[both][:, None, :], axis=2)
    dist = np.where(np.arange(nb)[None, :] < d["n_roots"][both][:, None], dist, np.inf)
    k = dist.argmin(1)
    ref = d["roots"][both][np.arange(both.sum()), k]
    err = assert_mixed(g_x[both], ref, TOL, f"{tag} roots")
    multi = (d["n_roots"][both] > 1).mean() if both.any() else 0.0
    print(f"{tag}: S={S} valid={ov.mean():.4f} flips={len(flips)} multi-root={multi:.4f} max root err={err:.2e}")
    return g_x, g_b


def test_deform_tiny_forward_samples(orc):
    w = synth.tiny_forward()
    m = orc.march(w.rays_o, w.rays_d, w.occ, w.occ_aabb, w.dt, w.n_per_ray, w.max_steps)
    _deform_check(orc, w, m["xs"].astype(np.float32), "tiny")


def test_deform_identity_pose():
    K = _K()
    w = synth.tiny_forward()
    xp = synth.random_points(1000, 7)
    Dz, Dy, Dx, nb = w.W.shape
    xc = torch.zeros(3, 1000, device=dev())
    bone = torch.zeros(1000, dtype=torch.int16, device=dev())
    steps = torch.zeros(1000, dtype=torch.int16, device=dev())
    ws = torch.empty(K.deform_workspace_size(Dx, Dy, Dz), dtype=torch.uint8, device=dev())
    K.snarf_deform(soa(xp), 1000, 1000, up(synth.identity_pose().astype(np.float32)), up(w.W), w.skin_aabb,
                   w.hash_aabb, 10, 1e-6, 1e-5, xc, bone, None, steps, ws)
    torch.cuda.synchronize()
    assert (host(bone) == 0).all()
    assert (host(steps) == 0).all()
    np.testing.assert_array_equal(host(xc).T, xp.astype(np.float64))


def test_deform_train_pose_ragged(orc):
    w = synth.train_step()
    rng = np.random.default_rng(3)
    xt = np.c_[rng.uniform(0.1, 0.9, 4099), rng.uniform(0.1, 0.9, 4099), rng.uniform(0.3, 0.7, 4099)]
    xp = indep.lbs_scipy(w.B, w.W, w.skin_aabb)(xt).astype(np.float32)
    _deform_check(orc, w, xp, "train pose")


@pytest.mark.parametrize("S,count", [(1, None), (8, None), (9, None), (4099, None), (16384, None), (300, 129),
                                     (16384, 7), (16385, 16384)])
def test_deform_lanes_per_sample(S, count):
    """Calls of at most 16,384 samples take 32 lanes a sample, larger ones
    eight: the same bits for every sample in either, on ragged counts, under a
    device count and at the border; nothing past the count."""
    K = _K()
    w = synth.train_step()
    big = 16385 + 64
    Dz, Dy, Dx, _ = w.W.shape
    xp = synth.sample_posed_points(synth.make_skeleton(0), w.B.astype(np.float64), big, 13).astype(np.float32)
    xp[5] = [9.0, 9.0, 9.0]  # no root

    def run(n, cnt):
        xc = torch.full((3, n), -7.0, device=dev())
        bone = torch.full((n,), -7, dtype=torch.int16, device=dev())
        resid = torch.full((n,), -7.0, device=dev())
        steps = torch.full((n,), -7, dtype=torch.int16, device=dev())
        ws = torch.empty(K.deform_workspace_size(Dx, Dy, Dz), dtype=torch.uint8, device=dev())
        Sd = None if cnt is None else torch.tensor([cnt], device=dev())
        K.snarf_deform(soa(xp[:n]), n, n, up(w.B), up(w.W), w.skin_aabb, w.hash_aabb, 10, 1e-6, 1e-5, xc, bone, resid,
                       steps, ws, S_dev=Sd)
        torch.cuda.synchronize()
        return host(xc), host(bone), host(resid), host(steps)

    n = S if count is None else count
    for got, ref in zip(run(S, count), run(big, None)):
        assert got[..., :n].tobytes() == ref[..., :n].tobytes()
        assert (got[..., n:] == -7).all()


@pytest.mark.parametrize("nb", [1, 2, 3, 5, 8, 9, 16, 17, 24])
def test_deform_lanes_by_bones_and_count(nb):
    """The lanes per sample and the source of the corners go by the number of
    bones and of samples, on the device where the count is there: the same
    bits in all of them, nothing past the count."""
    K = _K()
    w = synth.train_step()
    big = 20000
    Dz, Dy, Dx, _ = w.W.shape
    W = np.ascontiguousarray(w.W[..., :nb] + np.float32(1e-3))
    W = (W / W.sum(-1, keepdims=True)).astype(np.float32)
    B = np.ascontiguousarray(w.B[:nb])
    xp = synth.sample_posed_points(synth.make_skeleton(0), w.B.astype(np.float64), big, 17).astype(np.float32)
    xp[5] = [9.0, 9.0, 9.0]  # no root
    ws = torch.empty(K.deform_workspace_size(Dx, Dy, Dz), dtype=torch.uint8, device=dev())

    def run(cap, cnt):
        xc = torch.full((3, cap), -7.0, device=dev())
        bone, steps = (torch.full((cap,), -7, dtype=torch.int16, device=dev()) for _ in range(2))
        Sd = None if cnt is None else torch.tensor([cnt], device=dev())
        K.snarf_deform(soa(xp[:cap]), cap, cap, up(B), up(W), w.skin_aabb, w.hash_aabb, 10, 1e-6, 1e-5, xc, bone, None,
                       steps, ws, S_dev=Sd)
        torch.cuda.synchronize()
        return host(xc), host(bone), host(steps)

    ref = run(big, None)
    assert (ref[1] >= 0).any()
    for cap, cnt in ((100, None), (2049, None), (6145, None), (16384, None), (big, 100), (big, 6145), (big, 16385)):
        n = cap if cnt is None else cnt
        for got, r in zip(run(cap, cnt), ref):
            assert got[..., :n].tobytes() == r[..., :n].tobytes(), (cap, cnt)
            assert (got[..., n:] == -7).all(), (cap, cnt)


@pytest.mark.parametrize("log2T,scale,tdt", [(14, 1e-4, "f32"), (19, 1e-4, "f32"), (19, 0.5, "f32"),
                                             (19, 0.5, "f16")])
def test_hash_encode(orc, log2T, scale, tdt):
    K = _K()
    S = 5003
    x = synth.random_points(S, 31)
    x[:4] = [[0, 0, 0], [1, 1, 1], [0.5, 0.5, 0.5], [1, 0, 1]]
    table = synth.make_hash_table(16, 1 << log2T, 2, seed=5, scale=scale).astype(np.float32)
    if tdt == "f16":
        table = table.astype(np.float16)
    bone = np.where(np.arange(S) % 7 == 3, -1, 2).astype(np.int16)
    feat = torch.empty(16 * S * 2, device=dev())
    K.hashgrid_encode(soa(x), up(bone), S, S, up(table), 16.0, 1.38, (0, 0, 0, 1, 1, 1), feat)
    torch.cuda.synchronize()
    got = host(feat).reshape(16, S, 2).transpose(1, 0, 2).reshape(S, 32)
    ref = orc.hash_encode(x, table, orc.resolutions(16), np.array([0, 0, 0, 1, 1, 1.0]), valid=bone)
    err = assert_mixed(got, ref, TOL, f"hash T=2^{log2T} scale={scale} {tdt}")
    assert (got[bone < 0] == 0).all()
    print(f"hash T=2^{log2T} scale {scale} {tdt}: max err {err:.2e}")


@pytest.mark.parametrize("L", [6, 12])
def test_hash_encode_level_counts(orc, L):
    """Level counts other than 16: with L <= 8 each XCD serves one level (a
    lane takes one level), with L = 12 XCDs 0-3 serve two levels and 4-7
    one (a lane's second level is past L)."""
    K = _K()
    S = 3001
    x = synth.random_points(S, 33)
    table = synth.make_hash_table(L, 1 << 16, 2, seed=8, scale=0.5).astype(np.float32)
    bone = np.where(np.arange(S) % 5 == 1, -1, 0).astype(np.int16)
    feat = torch.full((L * S * 2,), 9.0, device=dev())
    K.hashgrid_encode(soa(x), up(bone), S, S, up(table), 16.0, 1.38, (0, 0, 0, 1, 1, 1), feat)
    torch.cuda.synchronize()
    got = host(feat).reshape(L, S, 2).transpose(1, 0, 2).reshape(S, 2 * L)
    ref = orc.hash_encode(x, table, orc.resolutions(L), np.array([0, 0, 0, 1, 1, 1.0]), valid=bone)
    err = assert_mixed(got, ref, TOL, f"hash L={L}")
    assert (got[bone < 0] == 0).all()
    print(f"hash L={L}: max err {err:.2e}")


def test_hash_encode_two_samples_per_lane(orc):
    """A frame-sized capacity (2^22 samples, from which a lane takes two
    samples) with a device-side count of 3001: the counted samples match the
    oracle, the rest of the feature array is untouched."""
    K = _K()
    cap, S = 1 << 22, 3001
    x = synth.random_points(S, 34)
    xs = torch.zeros((3, cap), device=dev())
    xs[:, :S] = up(x.T, torch.float32)
    bone = torch.zeros(cap, dtype=torch.int16, device=dev())
    bone[:S] = up(np.where(np.arange(S) % 6 == 2, -1, 1).astype(np.int16))
    table = synth.make_hash_table(16, 1 << 19, 2, seed=10, scale=0.5).astype(np.float16)
    feat = torch.full((16, cap, 2), 5.0, device=dev())
    count = torch.tensor([S], dtype=torch.int64, device=dev())
    K.hashgrid_encode(xs, bone, cap, cap, up(table), 16.0, 1.38, (0, 0, 0, 1, 1, 1), feat, S_dev=count)
    torch.cuda.synchronize()
    got = host(feat[:, :S, :]).transpose(1, 0, 2).reshape(S, 32)
    valid = host(bone[:S])
    ref = orc.hash_encode(x, table, orc.resolutions(16), np.array([0, 0, 0, 1, 1, 1.0]), valid=valid)
    err = assert_mixed(got, ref, TOL, "hash two samples per lane")
    assert (got[valid < 0] == 0).all()
    assert bool((feat[:, S:, :] == 5.0).all())
    print(f"hash two samples per lane: max err {err:.2e}")


@pytest.mark.parametrize("S,L,cap", [(1, 16, 1), (257, 16, 257), (7 * 256, 12, 7 * 256), (8 * 256 + 1, 16, 8 * 256 + 1),
                                     (11 * 256 + 5, 20, 11 * 256 + 5), (5 * 256 + 3, 16, 1 << 15), (0, 16, 4096)])
def test_hash_encode_fp16_level_turns(orc, S, L, cap):
    """FP16 table: the level pairs change XCD with the chunk slot.  Fewer than
    eight chunks, eight and more, two level groups, and a device-side count of
    fewer chunks than the capacity has slots: every level of every sample is
    written once (the oracle's values), nothing past the count."""
    K = _K()
    x = synth.random_points(max(S, 1), 35)[:S]
    xs = torch.zeros((3, cap), device=dev())
    if S:
        xs[:, :S] = up(x.T, torch.float32)
    table = synth.make_hash_table(L, 1 << 14, 2, seed=11, scale=0.5).astype(np.float16)
    feat = torch.full((L, cap, 2), 5.0, device=dev())
    count = torch.tensor([S], dtype=torch.int64, device=dev()) if cap > S else None
    K.hashgrid_encode(xs, None, cap, cap, up(table), 16.0, 1.38, (0, 0, 0, 1, 1, 1), feat, S_dev=count)
    torch.cuda.synchronize()
    assert bool((feat[:, S:, :] == 5.0).all())
    if S:
        got = host(feat[:, :S, :]).transpose(1, 0, 2).reshape(S, 2 * L)
        ref = orc.hash_encode(x, table, orc.resolutions(L), np.array([0, 0, 0, 1, 1, 1.0]))
        assert_mixed(got, ref, TOL, f"hash level turns S={S} L={L}")


@pytest.mark.parametrize("S,L", [(1, 20), (4 * 256, 20), (4 * 256 + 1, 20), (3 * 256 - 1, 16), (256, 32)])
def test_hash_encode_fp16_counts_and_groups(orc, S, L):
    """Device-side counts that end at, before and after a chunk, with one or
    two level groups: slots without a chunk leave, the others write all."""
    test_hash_encode_fp16_level_turns(orc, S, L, 1 << 14)


def test_hash_encode_bf16_features(orc):
    K = _K()
    S = 2049
    x = synth.random_points(S, 32)
    table = synth.make_hash_table(16, 1 << 19, 2, seed=5, scale=0.5).astype(np.float16)
    feat = torch.empty(16 * S * 2, dtype=torch.bfloat16, device=dev())
    K.hashgrid_encode(soa(x), None, S, S, up(table), 16.0, 1.38, (0, 0, 0, 1, 1, 1), feat)
    torch.cuda.synchronize()
    got = host(feat).reshape(16, S, 2).transpose(1, 0, 2).reshape(S, 32)
    ref = orc.hash_encode(x, table, orc.resolutions(16), np.array([0, 0, 0, 1, 1, 1.0]))
    # BF16 storage of the FP32 result: half an ulp of an 8-bit significand,
    # relative to max(|ref|, 1e-3) (the FP32 interpolation error is ~1e-7)
    assert_mixed(got, ref, 2 ** -8, "hash bf16 features", scale=1e-3)


def _feat_tensor(feat_rows, dtype=torch.float32):
    S = feat_rows.shape[0]
    return up(feat_rows.reshape(S, 16, 2).transpose(1, 0, 2).reshape(-1), dtype)


@pytest.mark.parametrize("S", [1, 15, 16, 1000, 4099])
def test_mlp_fwd_f32(orc, S):
    K = _K()
    rng = np.random.default_rng(S)
    feat = rng.normal(0, 0.5, (S, 32)).astype(np.float32)
    params = synth.make_mlp(seed=3, sigma_bias=0.5).astype(np.float32)
    bone = np.where(rng.uniform(size=S) < 0.1, -1, 0).astype(np.int16)
    ld = S + 5
    sigma = torch.empty(S, device=dev())
    rgb = torch.zeros(3, ld, device=dev())
    K.mlp_fwd(feat_dev(feat, ld), up(bone), S, ld, up(params), K.F32, sigma, rgb)
    torch.cuda.synchronize()
    s_ref, c_ref = orc.mlp_fwd(feat, params, valid=bone)
    assert_mixed(host(sigma), s_ref, TOL, "sigma")
    assert_mixed(host(rgb[:, :S]).T, c_ref, TOL, "rgb")


def test_mlp_fwd_bf16(orc):
    K = _K()
    S = 4099
    rng = np.random.default_rng(9)
    feat = rng.normal(0, 0.5, (S, 32)).astype(np.float32)
    params = synth.make_mlp(seed=3).astype(np.float32)
    sigma = torch.empty(S, device=dev())
    rgb = torch.zeros(3, S, device=dev())
    fb = _feat_tensor(feat, torch.bfloat16)
    K.mlp_fwd(fb, None, S, S, up(params), K.BF16, sigma, rgb)
    torch.cuda.synchronize()
    feat_b = host(fb).reshape(16, S, 2).transpose(1, 0, 2).reshape(S, 32)
    # (1) the oracle's BF16 storage form (weights and hidden activations
    # stored as bfloat16, ReLU decided on them, as the kernel does): the
    # kernel differs only by its FP32 accumulation, which can move a stored
    # activation by one bfloat16 step where its FP32 value sits on a rounding
    # boundary.  Every output within 2^-8 of the sum of its products'
    # magnitudes (any such steps), and 99 % of the samples within 1e-5 of it
    from tests import bounds
    s_q, c_q = orc.mlp_fwd(feat_b, params, bf16=True)
    om = bounds.mlp_fwd_magnitude(np.abs(feat_b), params)
    d_o = np.abs(np.log(np.maximum(host(sigma), 1e-300)) - np.log(s_q)) / om[:, 0]
    d_c = (np.abs(host(rgb).T - c_q) / om[:, 1:]).max(1)
    worst = np.maximum(d_o, 4 * d_c)  # |dc| <= |do| / 4
    assert worst.max() <= 2.0 ** -8, worst.max()
    assert np.quantile(worst, 0.99) <= 1e-5, np.quantile(worst, 0.99)
    # (2) reported: the oracle in FP64 on the BF16-rounded inputs and weights
    params_b = host(up(params).bfloat16())
    s_ref, c_ref = orc.mlp_fwd(feat_b, params_b)
    e_s = np.abs(host(sigma) - s_ref) / np.maximum(1, s_ref)
    e_c = np.abs(host(rgb).T - c_ref)
    print(f"bf16 mlp vs storage-form oracle: max {worst.max():.2e}, p99 {np.quantile(worst, 0.99):.2e} of the "
          f"magnitude; vs FP64 on rounded weights: sigma mean {e_s.mean():.2e} max {e_s.max():.2e}; "
          f"rgb mean {e_c.mean():.2e} max {e_c.max():.2e}")
    assert e_c.mean() < 1e-3 and e_s.mean() < 2e-3


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("S,cap", [(1, 1), (65, 80), (131100, 131107), (0, 70)])
def test_mlp_fwd_ragged(orc, S, cap, dtype):
    """Ragged ends of the 16-sample tiles and of the waves' rounds, with
    padding rows, invalid samples and a device count below the capacity.
    Features, weights and biases are small multiples of powers of two, so the
    hidden layers are exact and both sides store the same activations; the
    outputs differ by the FP32 sums of 65 terms (each rounding at most 2^-24
    of the terms' magnitudes) and a few roundings of the exponential."""
    from tests import bounds
    K = _K()
    rng = np.random.default_rng(S + 9)
    ld = cap + 3
    feat = np.full((cap, 32), np.nan, np.float32)  # past the count: not to be used
    feat[:S] = rng.integers(-8, 9, (S, 32)) / 8
    params = np.concatenate([rng.integers(-4, 5, k) / q for k, q in
                             [(2048, 16), (64, 8), (4096, 64), (64, 8), (256, 16), (4, 8)]]).astype(np.float32)
    bone = np.where(rng.uniform(size=cap) < 0.2, -1, 1).astype(np.int16)
    b16 = dtype == "bf16"
    sigma, rgb = torch.full((ld,), 9.0, device=dev()), torch.full((3, ld), 9.0, device=dev())
    Sd = None if cap == S else torch.tensor([S], dtype=torch.int64, device=dev())
    K.mlp_fwd(feat_dev(feat, ld, torch.bfloat16 if b16 else torch.float32), up(bone), cap, ld, up(params),
              K.BF16 if b16 else K.F32, sigma, rgb, S_dev=Sd)
    torch.cuda.synchronize()
    assert (host(sigma)[S:] == 9.0).all() and (host(rgb)[:, S:] == 9.0).all()
    if S == 0:
        return
    s_ref, c_ref = orc.mlp_fwd(feat[:S], params, valid=bone[:S], bf16=b16)
    om = 70 * 2.0 ** -24 * bounds.mlp_fwd_magnitude(np.abs(feat[:S]), params)
    es, ec = np.abs(host(sigma)[:S] - s_ref), np.abs(host(rgb)[:, :S].T - c_ref)
    assert (es <= s_ref * (om[:, 0] + 2.0 ** -21)).all()
    assert (ec <= om[:, 1:] / 4 + 2.0 ** -22).all()


def test_volrender_fwd(orc):
    K = _K()
    w = synth.train_step()
    w = synth.ray_subset(w, np.arange(0, w.R, 2))
    m = orc.march(w.rays_o, w.rays_d, w.occ, w.occ_aabb, w.dt, w.n_per_ray, w.max_steps)
    S = m["xs"].shape[0]
    rng = np.random.default_rng(0)
    sig = rng.uniform(0, 60, S).astype(np.float32)
    sig[::17] = 0
    rgb = rng.uniform(0, 1, (S, 3)).astype(np.float32)
    R = w.R
    for thr in (0.0, 1e-4, 0.3):
        color = torch.empty(R, 3, device=dev())
        opac = torch.empty(R, device=dev())
        n_used = torch.empty(R, dtype=torch.int32, device=dev())
        Tf = torch.empty(R, device=dev())
        K.volrender_fwd(up(sig), soa(rgb), S, up(m["ray_off"]), up(m["ray_dt"], torch.float32), R, thr, color, opac,
                        n_used, Tf)
        torch.cuda.synchronize()
        ref = orc.composite_fwd(sig, rgb, m["ray_off"], m["ray_dt"].astype(np.float32), thr)
        nu = host(n_used)
        same = nu == ref["n_used"]
        assert same.mean() > 0.999, thr
        assert_mixed(host(color)[same], ref["color"][same], TOL, f"color thr={thr}")
        assert_mixed(host(opac)[same], ref["opacity"][same], TOL, f"opacity thr={thr}")
        assert_mixed(host(Tf)[same], ref["T_final"][same], TOL, f"T_final thr={thr}")


def test_forward_end_to_end_tiny(orc):
    from paper_2212_10550_amd.pipeline import Pipeline
    w = synth.tiny_forward()
    p = Pipeline(w)
    S = p.forward()
    torch.cuda.synchronize()
    f = orc.forward(w, details=True)
    assert S == f["march"]["xs"].shape[0]
    gb = host(p.bone[:S]).astype(int)
    ob = f["deform"]["bone"]
    flip = (gb >= 0) != (ob >= 0)
    bad_rays = np.unique(f["march"]["ray_id"][flip])
    ok = np.ones(w.R, bool)
    ok[bad_rays] = False
    assert ok.mean() > 0.99
    err_c = assert_mixed(host(p.color)[ok], f["color"][ok], TOL, "pixel colour")
    err_a = assert_mixed(host(p.opacity)[ok], f["opacity"][ok], TOL, "opacity")
    print(f"tiny e2e: S={S}, flipped samples {flip.sum()}, rays compared {ok.sum()}, colour err {err_c:.2e}, "
          f"opacity err {err_a:.2e}")
