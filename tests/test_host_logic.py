"""Host-side logic of the binding and the library's size functions (no GPU:
the checks run before any device call)."""
import numpy as np
import pytest
import torch

from paper_2212_10550_amd import lib as K


def test_occ_words_is_whole_bricks():
    for G in (1, 7, 8, 16, 37, 128, 2048):
        nb, nbz = -(-G // 8), -(-G // 16)
        assert K.occ_words(G) == nb * nb * nbz * 32
    assert K.occ_words(0) == 0 and K.occ_words(2049) == 0
    assert K.occ_words(128) == (128 ** 3) // 32  # no padding at multiples of 16


def test_march_workspace_covers_masks_and_scan():
    for R, steps in ((1, 1), (8192, 128), (291600, 128), (1166400, 128), (1000, 300), (65535, 128), (65536, 128)):
        nblk = -(-R // (16 if R >= 65536 else 4))  # rays per workgroup: 4 per wave from 65536 rays, else 1
        need = 8 * nblk + 8 * (-(-nblk // 4096)) + 8 * R * (-(-steps // 64)) + 4 * R
        assert K.march_workspace_size(R, steps) >= need
    assert K.march_workspace_size(-1, 128) == 0 and K.march_workspace_size(10, -1) == 0


def test_march_workspace_never_falls():
    """A workspace sized for the largest call of a pool (the batch renderer's
    slots) holds every smaller one."""
    rays = sorted([0, 1, 5, 4096, 62500, 70001, 1 << 21, 1 << 24] +
                  [b + d for b in (32768, 65536, 131072, 524288) for d in (-17, -1, 0, 1, 300)])
    steps = (0, 1, 64, 65, 128, 1 << 22, (1 << 22) + 1)
    size = [[K.march_workspace_size(R, n) for n in steps] for R in rays]
    for i in range(len(rays)):
        for j in range(len(steps)):
            assert i == 0 or size[i][j] >= size[i - 1][j], (rays[i - 1], rays[i], steps[j])
            assert j == 0 or size[i][j] >= size[i][j - 1], (rays[i], steps[j - 1], steps[j])


def test_backward_and_regulariser_workspaces():
    assert K.hashgrid_encode_bwd_workspace_size(36503, 16) >= 4 * 3 * 16 * 36503
    assert K.hashgrid_encode_bwd_workspace_size(-1, 16) == 0
    # binned table gradient: 12-byte records, 8 per sample and level, dominate
    n = K.hashgrid_table_grad_workspace_size(36503, 16, 1 << 19)
    assert 12 * 8 * 16 * 36503 <= n < 12 * 8 * 16 * 36503 + (8 << 20)
    assert K.hashgrid_table_grad_workspace_size(36503, 16, 1 << 22) > 0  # 16384 tiles of 4096 entries
    assert K.hashgrid_table_grad_workspace_size(36503, 16, 1 << 23) == 0  # beyond the tile limit
    assert K.hashgrid_table_grad_workspace_size(1 << 26, 16, 1 << 19) == 0  # 8 L S >= 2^32 records
    with pytest.raises(ValueError):
        K.hashgrid_table_grad_workspace_size(100, 16, 3 << 18)
    assert K.density_reg_workspace_size(10 ** 6) >= 4 * min(-(-10 ** 6 // 256), 1024)
    assert K.occgrid_build_workspace_size(64, 16, 2, K.F32, 64, 64, 32) >= 64 ** 3 * (12 + 12 + 4 + 12 + 2 + 128)
    assert K.occgrid_build_workspace_size(257, 16, 2, K.F32, 64, 64, 32) == 0
    assert K.occgrid_build_workspace_size(64, 16, 2, K.BF16, 64, 64, 32) < \
        K.occgrid_build_workspace_size(64, 16, 2, K.F32, 64, 64, 32)


def test_binding_rejects_bad_shapes_before_any_device_call():
    cpu = torch.zeros
    with pytest.raises(ValueError):
        K.occ_pack(cpu(4, 4, 5, dtype=torch.uint8), cpu(64, dtype=torch.int32))
    with pytest.raises(ValueError):
        K.occ_pack(cpu(16, 16, 16, dtype=torch.uint8), cpu(10, dtype=torch.int32))
    with pytest.raises(ValueError):
        K.adam(cpu(10), cpu(9), cpu(10), cpu(10), 1e-2)
    with pytest.raises(ValueError):
        K.occ_from_density(cpu(100), 8, 0.5, 1, cpu(K.occ_words(8), dtype=torch.int32))
    # shapes fine, but host tensors: refused by the pointer check
    with pytest.raises(TypeError):
        K.adam(cpu(10), cpu(10), cpu(10), cpu(10), 1e-2)


def test_flags_are_distinct_bits():
    flags = [K.OVERWRITE, K.TABLE_COARSE, K.TABLE_FINE]
    assert all(f & (f - 1) == 0 for f in flags) and len(set(flags)) == 3


def test_autograd_front_end_dtype_checks():
    from paper_2212_10550_amd import autograd as A
    cfg = A.HashConfig(16.0, 1.38, (0, 0, 0, 1, 1, 1))
    with pytest.raises(TypeError):
        A.hash_encode(torch.zeros(3, 4), torch.zeros(4, dtype=torch.int16), torch.zeros(16, 64, 2).half(), cfg)
    with pytest.raises(TypeError):
        A.mlp(torch.zeros(16, 4, 2).bfloat16(), torch.zeros(4, dtype=torch.int16), torch.zeros(6532))


def test_fork_and_join_when_streams_are_one(monkeypatch):
    """The pool hands a stream out again and again: a renderer's or a step's
    side stream may be the stream that the work is captured on.  No stream
    waits for itself, every other fork and join is there, and each pose runs."""
    import torch
    from paper_2212_10550_amd.batch import BatchRenderer
    from paper_2212_10550_amd.pipeline import Pipeline
    log = []

    class Stream:
        def __init__(self, n):
            self.n = n

        def __eq__(self, o):
            return self.n == o.n

        def __ne__(self, o):
            return self.n != o.n

        def wait_stream(self, o):
            log.append(("wait", self.n, o.n))

        def __enter__(self):
            log.append(("on", self.n))

        def __exit__(self, *a):
            pass

    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: Stream(2))
    monkeypatch.setattr(torch.cuda, "stream", lambda s: s)
    r = BatchRenderer.__new__(BatchRenderer)
    r.graph = r.persistent = None
    r.poses, r.assign = list("abcd"), [[0], [1], [2], [3]]
    r.slots = [type("Slot", (), {"stream": Stream(n)})() for n in (1, 2, 3, 4)]
    r._pose_forward = lambda sl, p: log.append(("pose", p))
    r.render()
    waits = [e for e in log if e[0] == "wait"]
    assert waits == [("wait", n, 2) for n in (1, 3, 4)] + [("wait", 2, n) for n in (1, 3, 4)]
    assert [e[1] for e in log if e[0] == "pose"] == list("abcd")

    for mode, sides in (("binned", (2, 3)), ("atomic", (2, 3)), ("atomic", (1, 2))):
        log.clear()
        p = Pipeline.__new__(Pipeline)
        p.table_grad_mode, p.timer, p._table_zeroed = mode, None, False
        p.side, p.side2 = Stream(sides[0]), Stream(sides[1])
        p.stages = lambda S, Sd: [(n, lambda n=n: log.append(("stage", n)))
                                  for n in ("loss+render_bwd", "mlp_bwd", "hash_bwd_x", "deform_bwd")]
        p._mark = lambda name: None
        p._table_grad = lambda S, Sd, **kw: log.append(("stage", "table"))
        p.backward(8)
        waits = [e for e in log if e[0] == "wait"]
        assert all(a != b for _, a, b in waits)
        assert len([e for e in log if e == ("stage", "table")]) == (1 if mode == "binned" else 2)
        if mode == "atomic":
            other = 3 if sides == (2, 3) else 1  # the side stream that is not the current one
            assert ("wait", other, 2) in waits and ("wait", 2, other) in waits
