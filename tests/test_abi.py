"""The C ABI library loads, exports every symbol include/lbm.h declares, and
its struct layouts match the Python binding.  No GPU is touched: only
host-side entry points (argument validation, sizes, strings) are called."""
import ctypes
import os
import re
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "lbm.h")


@pytest.fixture(scope="module")
def L():
    from paper_0704_0043_amd import lbm
    if not os.path.exists(lbm.LIB_PATH):
        from paper_0704_0043_amd import build
        build.build()
    return lbm


def declared_functions():
    text = open(HEADER).read()
    return sorted(set(re.findall(r"LBM_API\s+[\w\s\*]+?\b(lbm_\w+)\s*\(", text)))


def test_header_declares_the_boundary():
    names = declared_functions()
    for required in ("lbm_create", "lbm_step", "lbm_moments", "lbm_entropy_stats", "lbm_destroy"):
        assert required in names


def test_library_exports_every_declared_symbol(L):
    lib = L.lib()
    for name in declared_functions():
        assert hasattr(lib, name), name
    assert set(declared_functions()) == set(L.SIGNATURES)


def test_only_the_c_abi_is_exported(L):
    out = subprocess.run(["nm", "-D", "--defined-only", L.LIB_PATH], capture_output=True, text=True, check=True)
    text_syms = {ln.split()[-1] for ln in out.stdout.splitlines() if " T " in ln}
    assert text_syms == set(declared_functions())


def c_layout():
    """sizeof/offsetof of the ABI structs as seen by a C compiler."""
    probe = r'''
#include <stdio.h>
#include <stddef.h>
#include "lbm.h"
#define OFF(T, f) printf(#T "." #f " %zu\n", offsetof(T, f))
int main(void) {
  printf("lbm_domain_desc %zu\n", sizeof(lbm_domain_desc));
  printf("lbm_run_desc %zu\n", sizeof(lbm_run_desc));
  printf("lbm_entropy_stats_t %zu\n", sizeof(lbm_entropy_stats_t));
  OFF(lbm_domain_desc, beta); OFF(lbm_domain_desc, delta_trim); OFF(lbm_domain_desc, rho_init);
  OFF(lbm_domain_desc, f_init); OFF(lbm_domain_desc, probe_y);
  OFF(lbm_run_desc, flags); OFF(lbm_run_desc, stream); OFF(lbm_run_desc, workspace_bytes);
  OFF(lbm_entropy_stats_t, step); OFF(lbm_entropy_stats_t, total_entropy); OFF(lbm_entropy_stats_t, n_fluid);
  return 0;
}
'''
    import tempfile
    with tempfile.TemporaryDirectory() as d:
        src = os.path.join(d, "probe.c")
        exe = os.path.join(d, "probe")
        open(src, "w").write(probe)
        subprocess.run(["gcc", "-std=c11", "-I", os.path.join(ROOT, "include"), src, "-o", exe], check=True)
        out = subprocess.run([exe], capture_output=True, text=True, check=True).stdout
    return dict(ln.rsplit(" ", 1) for ln in out.strip().splitlines())


def test_struct_layouts_match_binding(L):
    lay = {k: int(v) for k, v in c_layout().items()}
    for cls in (L.lbm_domain_desc, L.lbm_run_desc, L.lbm_entropy_stats_t):
        assert ctypes.sizeof(cls) == lay[cls.__name__], cls.__name__
    for key, val in lay.items():
        if "." in key:
            struct, fld = key.split(".")
            assert getattr(getattr(L, struct), fld).offset == val, key


def test_host_only_entry_points(L):
    assert L.lbm_abi_version() == 3
    assert L.lbm_beta_from_nu(1e-4) == pytest.approx(1 / (6e-4 + 1), rel=1e-15)
    assert "invalid" in L.lbm_strerror(L.LBM_EINVAL)
    n = L.lbm_workspace_bytes([L.Domain(nx=128, ny=64)], L.Run(storage=L.LBM_F32))
    # two FP32 population buffers of 9 planes at least
    assert n >= 2 * 9 * 128 * 64 * 4
    # entry points taking a context reject NULL without touching a device
    lib = L.lib()
    ms = (L.ctypes.c_double * 2)()
    assert lib.lbm_kernel_times(None, 4, ms) == L.LBM_EINVAL
    assert lib.lbm_step(None, 1) == L.LBM_EINVAL
    assert lib.lbm_tile_config(None, None, None, None) == L.LBM_EINVAL


@pytest.mark.parametrize("bad", [
    dict(beta=1.5), dict(beta=-0.1), dict(delta_trim=-1.0), dict(delta_median=float("nan")),
    dict(nx=0), dict(bc=1, nx=3, ny=10), dict(lattice=3), dict(lattice=1, bc=1),
    dict(lattice=2, bc=2), dict(qe=7), dict(rho0=0.0), dict(probe=(500, 1)),
    dict(limiter=8, ens_k=0.0), dict(limiter=16, ens_c=0.0), dict(limiter=4, delta_ens=-1.0),
    dict(limiter=16, ens_c=1.0, ens_k=0.25), dict(limiter=4, ens_c=float("inf")),
    dict(bc=1, nx=10, ny=10, probe=(0, 5)), dict(limiter=128), dict(collision=2), dict(collision=1, qe=0),
    dict(limiter=64 | 2, ds_form=1), dict(bc=3, nx=3, ny=10), dict(lattice=1, bc=3),
])
def test_invalid_descriptors_are_rejected_before_any_device_call(L, bad):
    kw = dict(nx=32, ny=16)
    kw.update(bad)
    with pytest.raises(L.LbmError) as e:
        L.lbm_workspace_bytes([L.Domain(**kw)], L.Run())
    assert e.value.code == L.LBM_EINVAL
    with pytest.raises(L.LbmError) as e:
        L.lbm_create([L.Domain(**kw)], L.Run())
    assert e.value.code == L.LBM_EINVAL


@pytest.mark.parametrize("dom,run", [
    (dict(limiter=1), dict()),                               # no median filter
    (dict(limiter=2 | 8, ens_k=0.5), dict()),                # an ensemble-dependent limiter
    (dict(limiter=2, collision=1, qe=1), dict()),            # ELBM
    (dict(lattice=1, ny=1, limiter=2), dict()),              # D1Q3
    (dict(limiter=2), dict(tile_x=248)),                     # the fused step already
])
def test_adaptive_runs_need_both_forms_of_the_step(L, dom, run):
    kw = dict(nx=32, ny=16)
    kw.update(dom)
    r = L.Run(flags=L.LBM_RUN_ADAPTIVE, **run)
    for call in (L.lbm_workspace_bytes, L.lbm_create):
        with pytest.raises(L.LbmError) as e:
            call([L.Domain(**kw)], r)
        assert e.value.code == L.LBM_EINVAL


def test_adaptive_workspace_holds_the_second_form(L):
    """the fused form's tables (and its partial slots at 4-row tiles) come on top"""
    d = [L.Domain(nx=300, ny=70, limiter=3)]
    plain = L.lbm_workspace_bytes(d, L.Run())
    adaptive = L.lbm_workspace_bytes(d, L.Run(flags=L.LBM_RUN_ADAPTIVE))
    assert adaptive > plain


def test_mixed_batches_are_rejected(L):
    with pytest.raises(L.LbmError):
        L.lbm_workspace_bytes([L.Domain(qe=0), L.Domain(qe=1)], L.Run())
    with pytest.raises(L.LbmError):
        L.lbm_workspace_bytes([L.Domain(), L.Domain()], L.Run(tile_x=96))
    with pytest.raises(L.LbmError):
        L.lbm_workspace_bytes([L.Domain()], L.Run(tile_h=65))


# fake device addresses: these calls are refused on the host, before any
# device call, so the pointers are never used
F0, F1 = 1 << 20, 2 << 20


@pytest.mark.parametrize("bad", [
    dict(f0=0), dict(f1=0), dict(f1=F0), dict(n_steps=-1), dict(probe=(3, 3)),
    dict(f_init=np.ones(9 * 32 * 16)), dict(beta=2.0), dict(storage=7),
])
def test_static_entry_refuses_bad_arguments_on_the_host(L, bad):
    kw = dict(nx=32, ny=16, limiter=L.LBM_LIM_MEDIAN)
    call = dict(f0=F0, f1=F1, n_steps=1, storage=L.LBM_F32)
    for k in list(bad):
        if k in call:
            call[k] = bad.pop(k)
    kw.update(bad)
    with pytest.raises(L.LbmError) as e:
        L.lbm_step_static(L.Domain(**kw), call["storage"], call["f0"], call["f1"], call["n_steps"])
    assert e.value.code == L.LBM_EINVAL


def test_static_entry_refuses_domains_beyond_its_scratch(L):
    """4096^2 FP32 with the median filter needs its Delta S' plane (64 MiB)
    plus the work tables and partials: more than the static array."""
    d = L.Domain(nx=4096, ny=4096, limiter=L.LBM_LIM_MEDIAN | L.LBM_LIM_TRIM, ds_form=L.LBM_DS_QUADRATIC)
    with pytest.raises(L.LbmError) as e:
        L.lbm_step_static(d, L.LBM_F32, F0, F1, 1)
    assert e.value.code == L.LBM_ENOMEM
    assert str(L.LBM_STATIC_SCRATCH_BYTES) in str(e.value)
    # the same grid with trimming alone needs no plane: only n_steps = 0 is
    # safe to call without a GPU, and it is accepted
    L.lbm_step_static(L.Domain(nx=4096, ny=4096, limiter=L.LBM_LIM_TRIM), L.LBM_F32, F0, F1, 0)
    assert L.lib().lbm_step_static(None, 1, None, None, None, 1, None) == L.LBM_EINVAL


# sizes that have been taken ever since the entry exists: the largest tubes
# without and with the arrays of an ensemble limiter, the widest and the
# narrowest grids (n_steps = 0 returns before any device call)
@pytest.mark.parametrize("storage,dom", [
    (0, dict(lattice=1, nx=31_333_440, ny=1, limiter=0)),
    (1, dict(lattice=1, nx=31_333_440, ny=1, limiter=1)),
    (2, dict(lattice=1, nx=31_333_440, ny=1, limiter=2)),
    (0, dict(lattice=1, nx=3_699_040, ny=1, limiter=8, ens_k=0.5, delta_ens=0.1)),
    (1, dict(lattice=1, nx=6_612_096, ny=1, limiter=32, ens_c=0.1)),
    (1, dict(nx=64, ny=168_400, limiter=2)),
    (0, dict(nx=64, ny=102_531, limiter=2)),
])
def test_static_entry_takes_the_sizes_it_took(L, storage, dom):
    L.lbm_step_static(L.Domain(ds_form=L.LBM_DS_QUADRATIC, **dom), storage, F0, F1, 0)
