"""Misplaced register copies in the compiled kernels (isa_check): the scan on
listings made for it, and on the built library.  On the GPU, the kernels that
had them: lanes that meet again after the two ways of the FP64 sine."""
import numpy as np
import pytest

import workloads as W
from helpers import gpu_solve
from paper_1803_01215_amd import build, hjpd, isa_check

HEAD = "0000000000001000 <kern>:\n"
JOIN = ["s_and_saveexec_b64 s[0:1], vcc", "s_cbranch_execz 4", "v_add_f64 v[2:3], v[2:3], v[4:5]"]


def _listing(*ops):
    """Disassembly text; a branch's operand is the index of the instruction it goes to."""
    out = []
    for i, t in enumerate(ops):
        tail = ""
        if "cbranch" in t:
            tail = " <kern+0x%x>" % (4 * int(t.split()[1]))
        out.append("\t%s%s// %012X:%s" % (t, " " * 8, 0x1000 + 4 * i, tail))
    return HEAD + "\n".join(out) + "\n"


@pytest.mark.parametrize("between,bad", [
    ([], False),                                                    # nothing before the restore
    (["s_mov_b32 s4, 0"], False),                                   # scalar only
    (["v_writelane_b32 v9, s4, 0", "v_readlane_b32 s4, v9, 0"], False),
    (["v_accvgpr_write_b32 a6, v1"], True),
    (["s_mov_b32 s4, 0", "v_mov_b32_e32 v1, v2"], True),
    (["scratch_store_dword off, v1, off offset:4"], True),
])
def test_scan(between, bad):
    ops = JOIN + ["v_mul_f64 v[2:3], v[2:3], v[4:5]"] + between + ["s_or_b64 exec, exec, s[0:1]", "s_endpgm"]
    assert bool(isa_check.scan(_listing(*ops))) == bad
    # the skipped part out of line: what follows the branch is the join
    ops = ["s_and_saveexec_b64 s[0:1], vcc", "s_cbranch_execnz %d" % (4 + len(between))] + between + [
        "s_or_b64 exec, exec, s[0:1]", "s_endpgm", "v_add_f64 v[2:3], v[2:3], v[4:5]", "s_branch 2"]
    assert bool(isa_check.scan(_listing(*ops))) == bad


def test_built_library_has_none():
    assert len(isa_check.code_objects(hjpd.LIB_PATH)) == len(build.INSTANCES) + 3
    assert isa_check.misplaced(hjpd.LIB_PATH, build.HIPCC) == {}


@pytest.mark.gpu
@pytest.mark.parametrize("family,tile,opt", [
    ("quadrotor12", (8, 4), dict()), ("quadrotor12", (64, 4), dict()), ("quadrotor12", (8, 4), dict(hopf=True)),
    ("cnorm10", (16, 4), dict(starts=2, restarts=1, sigma_inc=0.5)),
])
def test_a_point_of_huge_angles_among_others(family, tile, opt):
    """Two points of a batch whose sines take the reduction of large arguments,
    in groups beside points whose sines do not: every point gets its outputs,
    and the others the bits that they have without the two."""
    quad = family == "quadrotor12"
    w = (W.quadrotor12() if quad else W.cnorm10(61)).subset(np.arange(61))
    hi = tile[0] * tile[1]
    w.N = np.random.default_rng(2).integers(hi // 2, hi + 1, w.n).astype(np.int32)
    w.t = 0.02 * w.N if quad else w.t
    w.N_max = hi
    kw = dict(dtype="f64", tol=1e-30, max_iter=12, lanes_per_point=tile[0], nodes_per_lane=tile[1], **opt)
    base = gpu_solve(w, **kw)
    w.x = w.x.copy()
    huge = [5, 40]
    w.x[huge, 6 if quad else 0] = 1e12
    g = gpu_solve(w, **kw)
    assert np.all(g["iters"] > 0) and np.all((g["status"] >= 0) & (g["status"] <= 2))
    for i in range(w.n):
        if i in huge:
            assert np.array_equal(g["x_traj"][i, w.N[i]], w.x[i])  # x_N = x
            continue
        for k in ("iters", "status", "phi"):
            assert g[k][i] == base[k][i], (k, i)
        for k in ("x_traj", "p_traj"):
            assert np.array_equal(g[k][i, :w.N[i] + 1], base[k][i, :w.N[i] + 1]), (k, i)
