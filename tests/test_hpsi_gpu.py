"""H*psi on the GPU (dg_apply_H) against the oracle's plane-wave H (Eq. (1)), element by element."""
import dataclasses
import sys

import numpy as np
import pytest

import workloads as W
from oracle import planewave
from tests.gpu_util import need_torch_cuda, rel_err

pytestmark = pytest.mark.gpu

FP64_TOL = 1e-12   # relative to max |H x|; FFT rounding ~ eps log N
FP32_TOL = 5e-6


def _run(els, n_vec, prec, seed=1, elem=-1):
    torch = need_torch_cuda()
    from paper_2003_00407_amd import dgalb as D
    print(f"[hpsi] grids={[e.n for e in els]} n_vec={n_vec} prec={prec} elem={elem}", flush=True)
    E = D.Elements(els)
    rng = np.random.default_rng(seed)
    use = [k for k in range(len(els)) if elem < 0 or k == elem]
    xs = [rng.standard_normal((n_vec, els[k].npts)) for k in use]
    dt = torch.float64 if prec == D.DG_FP64 else torch.float32
    x = torch.tensor(np.concatenate([a.ravel() for a in xs]), dtype=dt, device="cuda")
    y = E.apply_H(x, n_vec, prec, elem=elem)
    torch.cuda.synchronize()
    yh = y.double().cpu().numpy()
    errs = []
    off = 0
    for i, k in enumerate(use):
        n = els[k].npts
        X = xs[i].T
        if prec == D.DG_FP32:
            X = X.astype(np.float32).astype(np.float64)
        ref = planewave.hpsi(els[k], X)
        got = yh[off:off + n * n_vec].reshape(n_vec, n).T
        off += n * n_vec
        errs.append(rel_err(got, ref))
    return max(errs)


def test_hpsi_c1_fp64_odd_ncols():
    assert _run(W.make_config("c1").elements, 5, 0) < FP64_TOL


def test_hpsi_slab_batch_fp64():
    assert _run(W.small_slab(), 12, 0) < FP64_TOL


def test_hpsi_slab_batch_fp32():
    assert _run(W.small_slab(), 12, 2) < FP32_TOL


def test_hpsi_single_element_mode():
    assert _run(W.small_slab(), 7, 0, elem=4) < FP64_TOL


@pytest.mark.parametrize("n", [(8, 8, 64), (12, 12, 24), (24, 24, 12), (32, 32, 48), (64, 64, 16)])
def test_hpsi_line_lengths(n):
    """Every supported line length (radix 2, 3, 4 paths), with wells, FP64 and FP32."""
    L = tuple(0.45 * x for x in n)
    rng = np.random.default_rng(sum(n))
    el = W._box_element(n, L, rng.uniform(0, 1, (3, 3)) * np.array(L), 4)
    assert _run([el], 3, 0) < FP64_TOL
    assert _run([el], 3, 2) < FP32_TOL


def test_hpsi_c2_full_size_elements_fp64():
    """Two elements of the 4x4 slab at full size (48x48x64, projectors)."""
    els = W.make_config("c2").elements[:2]
    assert _run(els, 4, 0) < FP64_TOL
    assert _run(els, 4, 2) < FP32_TOL


@pytest.mark.parametrize("prec", [0, 2])
@pytest.mark.parametrize("elem", [-1, 1])
@pytest.mark.parametrize("n_vec", [1, 4])
def test_hpsi_in_place_and_through_copies_agree(prec, elem, n_vec):
    """Disjoint caller buffers are read and written in place, overlapping ones go through
    the context's blocks: the same kernels, so the same bits, packed, with odd leading
    dimensions, and with y in x's own memory or in its gaps."""
    torch = need_torch_cuda()
    from paper_2003_00407_amd import dgalb as D
    els = W.small_slab(n_states=8)[:3]
    E = D.Elements(els)
    N, ne = els[0].npts, len(els) if elem < 0 else 1
    print(f"[hpsi] routes prec {prec} elem {elem} n_vec {n_vec}", flush=True)
    dt = torch.float64 if prec == D.DG_FP64 else torch.float32
    x = torch.tensor(np.random.default_rng(8).standard_normal(N * n_vec * ne), dtype=dt, device="cuda")
    y = E.apply_H(x, n_vec, prec, elem=elem)
    own = x.clone()
    E.apply_H(own, n_vec, prec, elem=elem, y=own)
    assert torch.equal(own, y)
    ld = 2 * N + 3                       # x in the first N values of a column, y in the last N
    both = torch.zeros(ld * n_vec * ne + N + 3, dtype=dt, device="cuda")
    cols = both[:ld * n_vec * ne].view(ne, n_vec, ld)
    cols[:, :, :N] = x.view(ne, n_vec, N)
    E.apply_H(both, n_vec, prec, elem=elem, ldx=ld, ldy=ld, y=both[N + 3:])
    assert torch.equal(cols[:, :, N + 3:], y.view(ne, n_vec, N))
    assert torch.equal(cols[:, :, :N], x.view(ne, n_vec, N))
    out = torch.zeros((N + 1) * n_vec * ne, dtype=dt, device="cuda")
    E.apply_H(both, n_vec, prec, elem=elem, ldx=ld, ldy=N + 1, y=out)
    assert torch.equal(out.view(ne, n_vec, N + 1)[:, :, :N], y.view(ne, n_vec, N))
    assert torch.count_nonzero(out.view(ne, n_vec, N + 1)[:, :, N:]).item() == 0


def _with_projectors(el, lens, rng):
    """el with projectors on random supports of the given lengths, grouped in runs of equal
    support: (support points, projectors sharing it) per entry of lens."""
    idx, val, ptr, gam = [], [], [0], []
    for n, count in lens:
        pts = np.sort(rng.choice(el.npts, size=n, replace=False)).astype(np.int32)
        for _ in range(count):
            idx.append(pts)
            val.append(rng.standard_normal(n) / np.sqrt(n))
            ptr.append(ptr[-1] + n)
            gam.append(rng.uniform(-1.0, 1.0))
    return dataclasses.replace(el, proj_ptr=np.array(ptr, dtype=np.int64), proj_idx=np.concatenate(idx),
                               proj_val=np.concatenate(val), gamma=np.array(gam))


@pytest.mark.parametrize("prec,tol", [(0, FP64_TOL), (2, FP32_TOL)])
@pytest.mark.parametrize("n_vec", [1, 8, 9, 17])
def test_hpsi_projector_shapes(n_vec, prec, tol):
    """Projector groups of one to four with supports around the 256-point steps and two
    steps in flight, points with no, few and many entries, and an element whose table of
    projectors is too large for 16 columns in LDS (456 and more)."""
    rng = np.random.default_rng(5)
    box = W._box_element((12, 12, 12), (8.0, 8.0, 8.0), rng.uniform(0.0, 8.0, size=(2, 3)), 16)
    els = [_with_projectors(box, [(1, 1), (255, 2), (256, 3), (257, 4), (511, 1), (512, 4), (513, 2), (1728, 4)], rng),
           _with_projectors(box, [(40, 4)] * 116 + [(700, 1)], rng)]
    assert els[1].n_proj == 465
    for some in (els[:1], els):
        assert _run(some, n_vec, prec) < tol


@pytest.mark.parametrize("shift", ["first_y_on_last_x", "ldx_above_ldy", "ldx_below_ldy"])
def test_hpsi_overlap_across_element_groups(shift):
    """Overlapping buffers whose overlap crosses element groups (a stream each): every
    group's x is read before any group's y is written.  The first element is small, so its
    group has finished while the second one's 184 MB of x are still being copied."""
    torch = need_torch_cuda()
    from paper_2003_00407_amd import dgalb as D
    els = [W._box_element((n, n, n), (0.4 * n,) * 3, np.array([[1.0, 1.0, 1.0]]), 80) for n in (12, 64)]
    n_vec = 88
    print(f"[hpsi] overlap across groups: {shift}", flush=True)
    E = D.Elements(els, n_streams=2)
    small, big = els[0].npts, els[1].npts
    gen = torch.Generator(device="cuda").manual_seed(3)
    if shift == "first_y_on_last_x":     # packed; y of the small element on the last columns of the big one's x
        total = (small + big) * n_vec
        ldx = ldy = 0
        x_at, y_at, size = 0, total - small * n_vec, 2 * total
    else:                                # one start, an element's blocks further apart in one than in the other
        a, b = big, big + small
        ldx, ldy = (b, a) if shift == "ldx_above_ldy" else (a, b)
        x_at = y_at = 0
        size = 2 * b * n_vec
    buf = torch.randn(size, dtype=torch.float64, device="cuda", generator=gen)
    nx = total if ldx == 0 else 2 * ldx * n_vec
    ny = total if ldy == 0 else 2 * ldy * n_vec
    x = buf[x_at:x_at + nx].clone()
    for _ in range(3):
        buf[x_at:x_at + nx] = x
        ref = E.apply_H(x, n_vec, ldx=ldx, ldy=ldy, y=buf[y_at:y_at + ny].clone())   # y's padding stays as it is
        E.apply_H(buf[x_at:x_at + nx], n_vec, ldx=ldx, ldy=ldy, y=buf[y_at:y_at + ny])
        assert torch.equal(buf[y_at:y_at + ny], ref)
