"""Labels over the runs of 64-node segments at the sizes where they can go wrong: rows of one node
to several segments, last segments of one, two, 32 and 33 nodes, tiles cut by the box, every
periodic wrap, and masks from empty to full, against a flood fill on the host; a mask that shares
memory with the labels; rows whose runs fill whole segments."""
import ctypes as C

import numpy as np
import pytest

from paper_1708_01608_amd import sc

pytestmark = pytest.mark.gpu


def _reference(mask, e):
    """Canonical labels (1 + smallest linear index) of a periodic mask [nz, ny, nx] by repeated
    minima over the lattice's neighbours and pointer jumping."""
    n = mask.size
    idx = np.arange(1, n + 1, dtype=np.int64).reshape(mask.shape)
    big = n + 1
    lab = np.where(mask, idx, big)
    while True:
        new = lab
        for ex, ey, ez in e[1:]:
            new = np.minimum(new, np.roll(lab, (-ez, -ey, -ex), (0, 1, 2)))
        new = np.where(mask, new, big)
        flat = np.append(new.reshape(-1), big)
        new = np.where(mask, flat[np.minimum(new - 1, n)], big)  # jump to the label's own label
        if np.array_equal(new, lab):
            return np.where(mask, lab, 0).astype(np.uint32).reshape(-1)
        lab = new


def _masks(shape, seed):
    rng = np.random.default_rng(seed)
    nz, ny, nx = shape
    yield "empty", np.zeros(shape, bool)
    yield "full", np.ones(shape, bool)
    for p in (0.05, 0.3, 0.6):
        yield f"random {p}", rng.random(shape) < p
    m = np.zeros(shape, bool)
    m[:, :, 0] = m[:, :, -1] = True  # joined only around the box in x
    yield "x faces", m
    m = np.zeros(shape, bool)
    m[::2, ::2, :] = True            # whole rows, runs over every segment
    yield "rows", m
    m = np.zeros(shape, bool)
    m[:, 0, ::3] = m[:, -1, 1::3] = True  # diagonal links around the box in y
    yield "y wrap", m


def _label(g, mask_ptr, labels):
    nc = C.c_int64(-1)
    rc = g._lib.sc_label_bubbles_noalloc(g._h, C.c_void_p(mask_ptr), C.c_void_p(labels.data_ptr()),
                                         C.byref(nc))
    assert rc == sc.SC_OK, g._lib.sc_last_error()
    return labels.cpu().numpy().view(np.uint32), nc.value


@pytest.mark.parametrize("q,shape", [
    (9, (1, 4, 4)), (9, (1, 300, 65)), (9, (1, 17, 66)), (9, (1, 260, 97)), (9, (1, 5, 128)),
    (9, (1, 40, 96)), (19, (4, 4, 4)), (19, (17, 5, 65)), (19, (5, 33, 130)), (19, (18, 16, 64)),
    (19, (33, 17, 31)), (19, (4, 6, 193)),
    (19, (130, 127, 65)),  # enough segments for several a wave
])
def test_labels_of_masks(q, shape):
    import torch

    nz, ny, nx = shape
    print(f"[gpu] labels q={q} {nx}x{ny}x{nz}", flush=True)
    g = sc.Sim(q=q, nx=nx, ny=ny, nz=nz, K=0)
    e, _ = sc.lattice(q)
    for name, mask in _masks(shape, 3):
        if mask.size > 1 << 20 and name in ("full", "random 0.6", "rows", "x faces"):
            continue  # minutes on the host
        ref = _reference(mask, e)
        m = torch.from_numpy(mask.astype(np.uint8).reshape(-1)).cuda()
        torch.cuda.synchronize()
        labels = torch.full((g.N,), -1, device="cuda", dtype=torch.int32)
        torch.cuda.synchronize()
        lab, nc = _label(g, m.data_ptr(), labels)
        assert np.array_equal(lab, ref), name
        assert nc == len(np.unique(ref[ref > 0])), name
        # the mask inside the labels' own memory, at its start and at its end
        for off in (0, 3 * g.N, 3 * g.N - 3):
            both = torch.full((4 * g.N,), 7, device="cuda", dtype=torch.uint8)
            both[off:off + g.N] = m
            torch.cuda.synchronize()
            lab, nc2 = _label(g, both.data_ptr() + off, both.view(torch.int32))
            assert np.array_equal(lab, ref) and nc2 == nc, (name, off)
        lab, nc3 = g.label_bubbles(mask)
        assert np.array_equal(lab, ref) and nc3 == nc, name


# boxes of up to 2^15 nodes take the pass in one launch behind the mask, larger ones kernel by
# kernel; the last two lie on either side
@pytest.mark.parametrize("q,shape", [
    (9, (1, 6, 4)), (9, (1, 130, 65)), (9, (1, 33, 200)), (19, (4, 4, 5)), (19, (9, 17, 66)),
    (19, (12, 11, 130)), (9, (1, 128, 256)), (9, (1, 129, 256)),
])
@pytest.mark.parametrize("p", [0.1, 0.35])
def test_pass_labels_and_bubbles(q, shape, p):
    """Labels, bubble counts and centroids of a pass on a random gas field (clusters wrap around
    the box): the integer sums are exact, so everything is equal."""
    nz, ny, nx = shape
    print(f"[gpu] pass q={q} {nx}x{ny}x{nz} p={p}", flush=True)
    rng = np.random.default_rng(11)
    mask = rng.random(shape) < p
    flat = np.flatnonzero(mask.reshape(-1))
    assert len(flat) > 0
    nodes = rng.choice(flat, size=min(40, len(flat)), replace=False)
    xyz = np.stack([nodes % nx, nodes // nx % ny, nodes // (nx * ny)], axis=1)
    g = sc.Sim(q=q, nx=nx, ny=ny, nz=nz, K=0, amp=0.0, film_max=1)
    g.seed_nuclei(xyz.astype(float), np.full(len(nodes), -1.0), np.zeros(len(nodes)), 0.0)
    g.set_equilibrium(np.where(mask, 0.2, 1.9))
    g.test_pass()
    e, _ = sc.lattice(q)
    ref = _reference(mask, e)
    assert np.array_equal(g.last_labels(), ref)
    comp, _ = g.nuclei(len(nodes))
    assert np.array_equal(comp, ref[nodes])
    got = g.bubbles()
    assert [b["label"] for b in got] == sorted(set(ref[nodes].tolist()))
    idx = np.arange(g.N)
    pos = (idx % nx, idx // nx % ny, idx // (nx * ny))
    dims = (nx, ny, nz)
    for b in got:
        at = ref == b["label"]
        lead = int(np.flatnonzero(comp == b["label"])[0])
        assert b["n"] == int(at.sum()) and b["nucleus"] == lead
        for c in range(2 if q == 9 else 3):
            h = dims[c] // 2
            d = (pos[c][at] - xyz[lead, c] + h) % dims[c] - h
            assert b["centroid"][c] == float(xyz[lead, c]) + float(d.sum()) / float(b["n"])
    # a second pass (the first one's bubbles leave the slot map) on the moved field
    g.set_equilibrium(np.where(np.roll(mask, (1, 2), (1, 2)), 0.2, 1.9))
    g.test_pass()
    assert np.array_equal(g.last_labels(), _reference(np.roll(mask, (1, 2), (1, 2)), e))
