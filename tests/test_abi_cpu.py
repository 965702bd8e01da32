"""C-ABI library: loads without a GPU, exports every declared symbol, validates arguments."""
import ctypes
import os
import re

import numpy as np
import pytest

import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _lib():
    from paper_2003_00407_amd import dgalb
    return dgalb


def test_header_symbols_exported():
    hdr = open(os.path.join(ROOT, "include", "dg_alb.h")).read()
    declared = set(re.findall(r"\b(dg_[a-z_A-Z]+)\s*\(", hdr))
    d = _lib()
    lib = ctypes.CDLL(d.LIB_PATH)
    for name in declared:
        assert hasattr(lib, name), f"{name} declared in dg_alb.h but not exported"
    assert declared == set(d.EXPORTED)


def test_status_strings():
    d = _lib()
    assert d.status_string(0) == "DG_OK"
    assert d.status_string(-2) == "DG_ERR_SHAPE"
    assert d.status_string(99) == "DG_UNKNOWN_STATUS"


def test_query_workspace_sizes():
    d = _lib()
    els = W.make_config("c1").elements
    b1 = d.query_workspace(els)
    assert b1 > 8 * 16 ** 3 * 12 * 8  # eight N x K FP64 blocks at least
    b2 = d.query_workspace(W.small_slab())
    assert b2 > b1


@pytest.mark.parametrize("degree,stride", [(1, 1), (16, 1), (16, 2), (13, 4), (6, 3), (4, 9), (17, 2)])
def test_query_workspace_counts_the_band_energy_blocks(degree, stride):
    """Behind the solver's blocks there is one per iterate that a band energy keeps (Y_k
    where a segment starts and the one before it), Y_m, H Y_m, and one segment's inside."""
    d = _lib()
    el = W.make_config("c1").elements[0]
    kept = {k for k in range(degree) if k % stride == 0 or ((k + 1) % stride == 0 and k + 1 < degree)}
    blocks = len(kept) + 2 + min(stride, degree) - 1
    K = el.n_states + W.guard_count(el.n_states)
    assert el.npts % 64 == 0 and K % 2 == 0
    more = d.query_workspace([el], max_cheb_degree=degree, ckpt_stride=stride) - d.query_workspace([el])
    assert more == blocks * el.npts * K * 8


@pytest.mark.parametrize("degree,stride,ok", [(19, 1, False), (18, 1, True), (18, 2, True), (64, 8, True),
                                              (30, 30, True), (4, 37, False), (2 ** 31 - 1, 1, False)])
def test_query_workspace_band_energy_limit(degree, stride, ok):
    """The limit on degree and stride: pairs, two results and a segment within 40."""
    d = _lib()
    el = W.make_config("c1").elements[0]
    if ok:
        assert d.query_workspace([el], max_cheb_degree=degree, ckpt_stride=stride) > 0
        return
    with pytest.raises(d.DGError) as e:
        d.query_workspace([el], max_cheb_degree=degree, ckpt_stride=stride)
    assert e.value.status == d.DG_ERR_ARG


def test_query_workspace_rejects_bad_input():
    d = _lib()
    el = W.make_config("c1").elements[0]
    import dataclasses
    bad = dataclasses.replace(el, n=(16, 16, 20))          # 20 not a supported line length
    with pytest.raises(d.DGError) as e:
        d.query_workspace([bad])
    assert e.value.status == d.DG_ERR_SHAPE
    bad = dataclasses.replace(el, elem_lo=(10, 0, 0), elem_n=(10, 16, 16))
    with pytest.raises(d.DGError) as e:
        d.query_workspace([bad])
    assert e.value.status == d.DG_ERR_ARG
    bad = dataclasses.replace(el, n_states=0)
    with pytest.raises(d.DGError):
        d.query_workspace([bad])
    bad = dataclasses.replace(el, n_states=85)              # J + guards > 88
    with pytest.raises(d.DGError) as e:
        d.query_workspace([bad])
    assert e.value.status == d.DG_ERR_SHAPE
    # projector indices must be ascending
    sl = W.small_slab()[0]
    idx = sl.proj_idx.copy()
    idx[1], idx[2] = idx[2], idx[1]
    with pytest.raises(d.DGError) as e:
        d.query_workspace([dataclasses.replace(sl, proj_idx=idx)])
    assert e.value.status == d.DG_ERR_ARG
    assert "ascending" in d.last_error()


def test_more_states_than_element_points_rejected():
    """J_k ALBs need |E_k| >= J_k grid points (else the restriction is rank deficient)."""
    import dataclasses
    d = _lib()
    el = W.free_electron_element(n_states=7)
    line = dataclasses.replace(el, elem_lo=(3, 5, 0), elem_n=(1, 1, 6))     # 6 points < 7 states
    with pytest.raises(d.DGError) as e:
        d.query_workspace([line])
    assert e.value.status == d.DG_ERR_SHAPE
    assert "exceeds" in d.last_error()
    ok = dataclasses.replace(el, elem_lo=(3, 5, 0), elem_n=(1, 1, 16))      # 16 points: accepted
    assert d.query_workspace([ok]) > 0


def test_too_many_projectors_rejected():
    import dataclasses
    d = _lib()
    base = W.make_config("c1").elements[0]
    for n_p, ok in ((480, True), (481, False)):
        el = dataclasses.replace(base, proj_ptr=np.arange(n_p + 1, dtype=np.int64),
                                 proj_idx=np.arange(n_p, dtype=np.int32), proj_val=np.full(n_p, 0.1),
                                 gamma=np.full(n_p, 0.01))
        if ok:
            assert d.query_workspace([el]) > 0
        else:
            with pytest.raises(d.DGError) as e:
                d.query_workspace([el])
            assert e.value.status == d.DG_ERR_SHAPE


def test_non_finite_inputs_rejected():
    import dataclasses
    d = _lib()
    el = W.make_config("c1").elements[0]
    v = el.v_eff.copy()
    v[123] = np.nan
    with pytest.raises(d.DGError) as e:
        d.query_workspace([dataclasses.replace(el, v_eff=v)])
    assert e.value.status == d.DG_ERR_NUMERIC
    sl = W.small_slab()[0]
    g = sl.gamma.copy()
    g[2] = np.inf
    with pytest.raises(d.DGError) as e:
        d.query_workspace([dataclasses.replace(sl, gamma=g)])
    assert e.value.status == d.DG_ERR_NUMERIC


def test_solve_params_layout_matches_header():
    """The ctypes mirror of dg_solve_params has the C layout (field offsets, size)."""
    d = _lib()
    P = d.SolveParams
    assert P.x0_dev.offset == 32 and P.graph_iters.offset == 40
    assert P.seed.offset == 48 and P.warm_start.offset == 56
    assert ctypes.sizeof(P) == 64


def test_struct_layouts_match_the_c_compiler(tmp_path):
    """Every ctypes mirror against offsetof/sizeof as gcc lays out the header's structs."""
    import shutil
    import subprocess
    if shutil.which("gcc") is None:
        pytest.skip("no gcc")
    d = _lib()
    mirrors = {"dg_solve_params": d.SolveParams, "dg_chefsi_params": d.ChefsiParams, "dg_mesh_desc": d.MeshDesc}
    lines = ["#include <stddef.h>", "#include <stdio.h>", '#include "dg_alb.h"', "int main(void) {"]
    for cname, py in mirrors.items():
        lines.append(f'  printf("{cname} size %zu\\n", sizeof({cname}));')
        for fname, _ in py._fields_:
            lines.append(f'  printf("{cname} {fname} %zu\\n", offsetof({cname}, {fname}));')
    lines += ["  return 0;", "}"]
    src = tmp_path / "layout.c"
    src.write_text("\n".join(lines) + "\n")
    exe = tmp_path / "layout"
    inc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include")
    subprocess.run(["gcc", "-std=c11", "-I", inc, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split("\n")
    for line in filter(None, out):
        cname, field, value = line.split()
        py = mirrors[cname]
        got = ctypes.sizeof(py) if field == "size" else getattr(py, field).offset
        assert got == int(value), f"{cname}.{field}: ctypes {got}, C {value}"


def test_null_context_calls_fail_cleanly():
    d = _lib()
    lib = d._lib
    assert lib.dg_apply_H(None, -1, 1, 0, None, 0, None, 0) == d.DG_ERR_ARG
    assert lib.dg_get_ritz(None, None, None) == d.DG_ERR_ARG
    assert lib.dg_solve_elements(None, None, None, None, None) == d.DG_ERR_ARG
    assert lib.dg_make_alb(None, None, None) == d.DG_ERR_ARG
    assert lib.dg_get_vectors(None, None) == d.DG_ERR_ARG
    assert lib.dg_density(None, None, None, 0, 0, None, None) == d.DG_ERR_ARG
    assert lib.dg_chefsi(None, None, 0, None, None, None, None, None, None, None, None, 0, None) == d.DG_ERR_ARG
    assert lib.dg_query_chefsi(None, 0, 1, None) == d.DG_ERR_ARG
    lib.dg_destroy(None)


def test_pack_initial_layout():
    d = _lib()
    els = W.small_slab()[:2]
    x0 = d.pack_initial(els, 10)
    g = W.guard_count(els[0].n_states)
    assert x0.size == sum(e.npts * (e.n_states + g) for e in els)
    assert np.array_equal(x0[: els[0].npts], W.initial_block(els[0].npts, els[0].n_states + g, 10)[0])


def test_destructor_at_interpreter_exit(monkeypatch):
    """A context still alive when the interpreter clears the module's globals is released
    once, without an error."""
    d = _lib()
    E = object.__new__(d.Elements)
    E.ctx = ctypes.c_void_p(16)
    calls = []
    E._destroy = lambda ctx: calls.append(ctx.value)
    with monkeypatch.context() as m:
        m.setattr(d, "C", None)
        E.__del__()
        E.__del__()
    assert calls == [16] and E.ctx.value is None
