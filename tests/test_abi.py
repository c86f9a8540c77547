"""C-ABI library checks that need no GPU: the built library loads, exports
every function include/vdsolve.h declares, and its host-only entry points
(defaults, sizing, status strings, argument validation) behave."""
import ctypes
import math
import os
import re
import subprocess
import sys

import pytest

from paper_2403_06654_amd import api

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "vdsolve.h")


def declared_functions():
    src = open(HEADER).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(vd_[a-z0-9_]+)\s*\(", src)))


def test_library_exports_every_declared_symbol():
    L = api.lib()
    names = declared_functions()
    assert len(names) >= 12
    for n in names:
        assert hasattr(L, n), n
    assert set(names) == set(api._SIGS), "binding and header disagree"


def test_one_hip_runtime_whichever_is_loaded_first():
    """The library opened before torch is imported must share torch's HIP runtime."""
    code = ("from paper_2403_06654_amd import api; api.lib(); import torch; "
            "print(len({l.split()[-1] for l in open('/proc/self/maps') if 'libamdhip64' in l}))")
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    assert int(r.stdout) == 1


def test_defaults():
    o = api.vd_solve_opts()
    api.lib().vd_default_opts(ctypes.byref(o))
    assert o.solver == api.VD_GMRES and o.restart == 30 and o.rtol == 1e-10
    assert o.precond == 1 and o.precision == api.VD_FP64 and math.isnan(o.rho0)
    assert o.max_iter == 2000 and o.inner_rtol == 1e-5 and o.max_outer == 10
    assert o.use_x0 == 0 and o.formulation == api.VD_FORM_L
    assert not o.history and o.history_cap == 0
    # the ABI struct layouts the binding mirrors (C: 8-byte alignment)
    assert ctypes.sizeof(api.vd_solve_opts) == 80 and ctypes.sizeof(api.vd_solve_info) == 48


def test_status_strings():
    for s in range(-7, 2):
        assert api.vd_status_string(s)
    assert api.vd_status_string(0) == "ok"


def test_workspace_bytes():
    wb = api.workspace_bytes
    c3 = wb((256, 256, 256))
    n = 256 ** 3
    # GMRES(30): 32 FP64 spectral vectors + operator work + b, x, tmp + coefficients
    assert c3 > 32 * n * 8 and c3 < 45 * n * 8
    assert wb((256, 256, 256), precision="fp32_refine") < c3
    assert wb((256, 256, 256), solver="cg") < c3
    assert wb((512, 512, 512)) > 7 * c3
    assert wb((1024, 1024)) > wb((128, 128)) * 50
    # the modified pressure form keeps -c (FP64 + FP32) and two spectral fields more
    assert wb((256, 256, 256), formulation="K") - c3 == n * (8 + 4) + 2 * n * 8
    assert wb((64, 64), formulation=7) == 0
    # invalid descriptors
    assert wb((100, 100)) == 0
    assert wb((8,)) == 0
    assert wb((2048,)) == 0
    d = api.make_desc((64, 64))
    d.length[0] = -1.0
    assert api.lib().vd_workspace_bytes(ctypes.byref(d), None) == 0


def test_workspace_bytes_helmholtz():
    """GMRES velocity solves on Fourier grids of two or three dimensions
    hold up to three systems' Krylov vectors at once; other solves one."""
    wb = api.workspace_bytes
    shape = (256, 256, 256)
    nspec = 256 * 256 * 128          # packed half spectrum (kx = 0 and nx/2 share slot 0)
    one = wb(shape)
    assert wb(shape, helmholtz_ncomp=1) == one
    extra = wb(shape, helmholtz_ncomp=2) - one
    # b, x, basis V_0..V_30, operator result and work: 35 FP64 spectral vectors (+ partials, state)
    assert 35 * nspec * 16 <= extra < 35 * nspec * 16 + (1 << 20)
    assert wb(shape, helmholtz_ncomp=3) - one == 2 * extra
    assert wb(shape, helmholtz_ncomp=7) == wb(shape, helmholtz_ncomp=3)
    e32 = wb(shape, helmholtz_ncomp=2, precision="fp32_refine") - wb(shape, precision="fp32_refine")
    assert 5 * nspec * 16 + 35 * nspec * 8 <= e32 < 5 * nspec * 16 + 35 * nspec * 8 + (1 << 20)
    assert wb((64, 128), helmholtz_ncomp=3) > wb((64, 128))
    # one system at a time: CG, RMR, 1D and Fourier-Chebyshev grids
    for kw in (dict(solver="cg"), dict(solver="rmr")):
        assert wb(shape, helmholtz_ncomp=3, **kw) == wb(shape, **kw)
    assert wb((512,), helmholtz_ncomp=3) == wb((512,))
    assert wb((65, 128), cheb=True, helmholtz_ncomp=3) == wb((65, 128), cheb=True)
    assert wb(shape, helmholtz_ncomp=0) == 0
    assert wb((100, 100), helmholtz_ncomp=3) == 0


def test_grid_create_rejects_bad_descriptors_without_touching_the_device():
    h = ctypes.c_void_p()
    for shape in [(100,), (8, 8), (4096,)]:
        d = api.make_desc(shape)
        assert api.lib().vd_grid_create(ctypes.byref(h), ctypes.byref(d), None) == -1
    d = api.make_desc((64,))
    d.ndim = 4
    assert api.lib().vd_grid_create(ctypes.byref(h), ctypes.byref(d), None) == -1
    d = api.make_desc((64,))
    d.basis[0] = 1
    assert api.lib().vd_grid_create(ctypes.byref(h), ctypes.byref(d), None) == -7
    assert api.lib().vd_grid_create(None, ctypes.byref(d), None) == -1


def test_null_handles_are_rejected():
    L = api.lib()
    assert L.vd_grid_destroy(None) == -1
    assert L.vd_set_density(None, None) == -1
    assert L.vd_apply_operator(None, 0, 0, 0.0, None, None) == -1
    assert L.vd_solve_pressure(None, None, None, None, None) == -1
    assert L.vd_solve_helmholtz(None, 1e-3, 1, None, None, None, None) == -1
    assert L.vd_profile_enable(None, 1) == -1


def test_build_flags_and_product_path_independent_of_oracle():
    # the product package never imports the oracle
    pkg = os.path.join(ROOT, "paper_2403_06654_amd")
    for dirpath, _, files in os.walk(pkg):
        for fn in files:
            if fn.endswith((".py", ".hip", ".cpp", ".hpp", ".h")):
                txt = open(os.path.join(dirpath, fn)).read()
                assert "import oracle" not in txt and "from oracle" not in txt, fn


def test_fractional_step_rejects_bad_parameters_without_touching_the_device():
    L = api.lib()
    h = ctypes.c_void_p()
    prm = api.vd_ns_params()
    L.vd_ns_default_params(ctypes.byref(prm))
    assert (prm.re, prm.sc, prm.visc_rtol, prm.pres_rtol, prm.restart) == (1.0, 1.0, 1e-12, 1e-12, 30)
    assert (prm.pres_solver, prm.pres_form) == (api.VD_GMRES, api.VD_FORM_L)
    for n in (8, 48, 1024):
        assert L.vd_ns_create(ctypes.byref(h), n, ctypes.byref(prm), None) == -1
    for field, bad in (("dt", 0.0), ("re", -1.0), ("s", -2.0), ("restart", 31), ("visc_rtol", 0.0),
                       ("pres_solver", 7), ("pres_form", 2)):
        p = api.vd_ns_params()
        L.vd_ns_default_params(ctypes.byref(p))
        setattr(p, field, bad)
        assert L.vd_ns_create(ctypes.byref(h), 32, ctypes.byref(p), None) == -1, field
    assert L.vd_ns_create(None, 32, None, None) == -1
    assert L.vd_ns_destroy(None) == -1
    assert L.vd_ns_step(None, 1, None) == -1
    assert L.vd_ns_errors(None, None) == -1
    assert L.vd_ns_init_taylor_green(None) == -1


def test_missing_library_fails_loudly(monkeypatch, tmp_path):
    """No fallback: without the built HIP library every entry point raises."""
    from paper_2403_06654_amd import api
    monkeypatch.setattr(api, "LIB_PATH", str(tmp_path / "libvdsolve.so"))
    monkeypatch.setattr(api, "_LIB", None)
    with pytest.raises(RuntimeError, match="is missing"):
        api.lib()
    with pytest.raises(RuntimeError, match="is missing"):
        api.vd_status_string(0)


def test_batch_entry_points_reject_bad_arguments():
    """Argument checks that need no device."""
    L = api.lib()
    assert L.vd_solve_pressure_batch(None, 2, None, None, None, None) == -1
    g = (ctypes.c_void_p * 1)()
    assert L.vd_solve_pressure_batch(g, 0, g, g, None, None) == -1
    assert L.vd_server_set_batch(None, 2) == -1
    srv = api.Server(hbm_budget=1 << 30, max_slots=1, dry_seconds=0.0)
    for bad in (0, 4):
        assert L.vd_server_set_batch(srv._h, bad) == -1
    assert L.vd_server_set_batch(srv._h, 1) == 0
    srv.close()

