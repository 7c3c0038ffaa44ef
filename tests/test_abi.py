"""The C ABI: symbols, defaults and argument checks.

CPU tests load librlsim.so and check that it exports every function
include/rlsim.h declares and rejects bad arguments that need no device.  GPU
tests cover the error paths that need a live handle.
"""
import ctypes
import os
import re
import subprocess

import numpy as np
import pytest

import workloads

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "rlsim.h")


def _declared():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(rlsim_[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    import paper_2207_07736_amd as p
    names = _declared()
    assert set(names) == set(p.EXPORTS), names
    lib = ctypes.CDLL(p.LIB_PATH)
    for name in names:
        assert hasattr(lib, name), name
    nm = subprocess.run(["nm", "-D", "--defined-only", p.LIB_PATH], capture_output=True, text=True, check=True).stdout
    exported = set(re.findall(r" T (rlsim_\w+)", nm))
    assert exported == set(names)
    assert "orc_" not in nm                      # the oracle is never linked in


def test_product_does_not_reach_the_oracle():
    pkg = os.path.join(ROOT, "paper_2207_07736_amd")
    for dirpath, _, files in os.walk(pkg):
        for f in files:
            if f.endswith((".py", ".hip", ".h", ".cpp")):
                text = open(os.path.join(dirpath, f)).read()
                assert "import oracle" not in text and "from oracle" not in text and "orc_" not in text, f


def test_cfg_default_matches_workload_constants():
    import paper_2207_07736_amd as p
    c = p.rlsim_cfg_default()
    for k, v in workloads.CARTPOLE.items():
        if k == "no_termination":
            assert c.flags == 0
            continue
        got = getattr(c, k)
        want = np.float32(v) if isinstance(v, float) else v
        assert np.float32(got) == want if isinstance(v, float) else got == want, k
    assert np.float32(c.theta_threshold_rad).view(np.uint32) == 0x3E567750
    assert c.stream is None


@pytest.mark.parametrize("n,words", [(0, 4), (1 << 30 | 1, 4), (16, 3), (16, 0), (1, (1 << 24) + 5), (1, 2**32 - 1)])
def test_create_rejects_bad_sizes(n, words):
    import paper_2207_07736_amd as p
    with pytest.raises(p.RlsimError) as e:
        p.rlsim_create(n, words)
    assert e.value.code == p.RLSIM_EINVAL
    assert p.rlsim_last_error(None)


@pytest.mark.parametrize("field,value", [("masscart", 0.0), ("half_length", -1.0), ("tau", float("nan")),
                                         ("reset_low", 1.0), ("gravity", float("inf"))])
def test_create_rejects_bad_cfg(field, value):
    import paper_2207_07736_amd as p
    c = p.rlsim_cfg_default()
    setattr(c, field, value)
    with pytest.raises(p.RlsimError) as e:
        p.rlsim_create(8, 4, c)
    assert e.value.code == p.RLSIM_EINVAL


def test_create_rejects_unknown_flags_and_null_out():
    import paper_2207_07736_amd as p
    c = p.rlsim_cfg_default()
    c.flags = 0x10
    with pytest.raises(p.RlsimError):
        p.rlsim_create(8, 4, c)
    assert p.lib.rlsim_create(8, 4, None, None) == p.RLSIM_EINVAL


def test_null_handle_calls():
    import paper_2207_07736_amd as p
    L = p.lib
    assert L.rlsim_destroy(None) == p.RLSIM_OK
    assert L.rlsim_reset(None, 0) == p.RLSIM_EINVAL
    assert L.rlsim_step_fused(None, 1, None, None) == p.RLSIM_EINVAL
    assert L.rlsim_get_state(None, None, None, None) == p.RLSIM_EINVAL
    assert L.rlsim_set_state(None, None, None, 0) == p.RLSIM_EINVAL
    L.rlsim_cfg_default(None)


# ---------------------------------------------------------------- GPU error paths
@pytest.mark.gpu
def test_state_and_argument_errors_with_handle():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2207_07736_amd as p
    sim = p.Simulator(300, 0, workloads.CARTPOLE)
    try:
        with pytest.raises(p.RlsimError) as e:
            sim.step(1)
        assert e.value.code == p.RLSIM_ESTATE
        with pytest.raises(p.RlsimError) as e:
            sim.get_state()
        assert e.value.code == p.RLSIM_ESTATE
        sim.reset(0)
        with pytest.raises(p.RlsimError) as e:
            sim.step(0)
        assert e.value.code == p.RLSIM_EINVAL
        tr = p.Trajectory(4, 300)
        bad = p.traj_struct(obs=tr.obs, action=tr.action)          # mixed NULLs
        with pytest.raises(p.RlsimError) as e:
            p.rlsim_step_fused(sim.h, 4, None, bad)
        assert e.value.code == p.RLSIM_EINVAL
        mis = p.rlsim_traj(tr.obs.data_ptr() + 2, tr.action.data_ptr(), tr.reward.data_ptr(), tr.done.data_ptr(),
                           None, None)
        with pytest.raises(p.RlsimError) as e:
            p.rlsim_step_fused(sim.h, 4, None, mis)
        assert e.value.code == p.RLSIM_EINVAL
        p0only = p.traj_struct(policy_p0=tr.obs)
        with pytest.raises(p.RlsimError) as e:
            p.rlsim_step_fused(sim.h, 4, None, p0only)
        assert e.value.code == p.RLSIM_EINVAL
        st, ep, t = sim.get_state()
        sim.set_state(st, ep, 2**32 - 5)
        sim.step(4)
        with pytest.raises(p.RlsimError) as e:
            sim.step(1)
        assert e.value.code == p.RLSIM_EINVAL
        with pytest.raises(p.RlsimError) as e:
            sim.set_state(None, None, 2**32)
        assert e.value.code == p.RLSIM_EINVAL
        # a failed call leaves the handle usable
        sim.set_state(None, None, 0)
        sim.step(4, tr.rows(0, 4))
        torch.cuda.synchronize()
        assert int(tr.action.max()) <= 1
        del tr
    finally:
        sim.close()


def test_create_rejects_zero_compute_factor():
    import paper_2207_07736_amd as p
    c = p.rlsim_cfg_default()
    assert c.compute_factor == 1
    c.compute_factor = 0
    with pytest.raises(p.RlsimError) as e:
        p.rlsim_create(8, 4, c)
    assert e.value.code == p.RLSIM_EINVAL


def test_binding_struct_layouts_match_the_header(tmp_path):
    """sizeof and every field offset of the three ABI structs, as a C compiler
    lays them out from include/rlsim.h, equal the ctypes binding's."""
    import paper_2207_07736_amd as p
    structs = {"rlsim_cfg": p.rlsim_cfg, "rlsim_traj": p.rlsim_traj, "rlsim_policy": p.rlsim_policy}
    lines = ['#include <stdio.h>', '#include <stddef.h>', '#include "rlsim.h"', "int main(void) {"]
    for name, cls in structs.items():
        lines.append(f'printf("{name} sizeof %zu\\n", sizeof({name}));')
        for field, _ in cls._fields_:
            lines.append(f'printf("{name} {field} %zu\\n", offsetof({name}, {field}));')
    lines.append("return 0; }")
    src = tmp_path / "layout.c"
    src.write_text("\n".join(lines))
    exe = tmp_path / "layout"
    subprocess.run(["gcc", "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe)], check=True)
    got = subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split("\n")
    for row in filter(None, got):
        name, field, val = row.split()
        cls = structs[name]
        want = ctypes.sizeof(cls) if field == "sizeof" else getattr(cls, field).offset
        assert int(val) == want, row


def test_probe_library_exports_and_rejects_bad_arguments():
    from paper_2207_07736_amd import probe
    text = re.sub(r"/\*.*?\*/", "", open(os.path.join(ROOT, "include", "rlsim_probe.h")).read(), flags=re.S)
    declared = set(re.findall(r"\b(rlsim_[a-z_]+)\s*\(", text))
    assert declared == set(probe.PROBE_EXPORTS)
    nm = subprocess.run(["nm", "-D", "--defined-only", probe.PROBE_LIB_PATH], capture_output=True, text=True,
                        check=True).stdout
    assert set(re.findall(r" T (rlsim_\w+)", nm)) == declared
    L = probe.probe_lib
    # rejected before any device call
    assert L.rlsim_probe_store(0, 4, 4, 4, 4, 4, None) == -1
    assert L.rlsim_probe_store(8, 0, 4, 4, 4, 4, None) == -1
    assert L.rlsim_probe_store(8, 1 << 23, 4, 4, 4, 4, None) == -1
    assert L.rlsim_probe_store((1 << 30) + 1, 4, 4, 4, 4, 4, None) == -1
    assert L.rlsim_probe_store(8, 4, None, 4, 4, 4, None) == -1
    assert L.rlsim_probe_store(8, 4, 6, 4, 4, 4, None) == -1     # misaligned obs
    assert L.rlsim_probe_policy_math(0, 0, 4, None) == -1
    assert L.rlsim_probe_policy_math(1, 1 << 32, 4, None) == -1
    assert L.rlsim_probe_policy_math(0, 16, None, None) == -1
    assert L.rlsim_probe_policy_math(0, 16, 6, None) == -1         # misaligned out_max
    assert L.rlsim_probe_stream(0, 16, 16, 16, None) == -1
    assert L.rlsim_probe_stream(4, None, 16, 16, None) == -1
    assert L.rlsim_probe_stream(4, 16, 24, 16, None) == -1          # misaligned a
    assert L.rlsim_probe_issue(10, 1, 1, 16, None, None) == -1         # unknown kind
    assert L.rlsim_probe_issue(0, 0, 1, 16, None, None) == -1
    assert L.rlsim_probe_issue(0, 1, 0, 16, None, None) == -1
    assert L.rlsim_probe_issue(5, 1, (1 << 19) + 1, 16, None, None) == -1
    assert L.rlsim_probe_issue(8, 1, (1 << 16) + 1, 16, None, None) == -1
    assert L.rlsim_probe_issue(9, 1, (1 << 16) + 1, 16, None, None) == -1
    assert L.rlsim_probe_issue(0, 1, 1, None, None, None) == -1
    assert L.rlsim_probe_issue(0, 1, 1, 18, None, None) == -1         # misaligned out
    assert L.rlsim_probe_issue(0, 1, 1, 16, 20, None) == -1           # misaligned clocks
    assert L.rlsim_probe_wall_clock_khz(None) == -1
    assert L.rlsim_probe_fill(0, 1, 16, None) == -1
    assert L.rlsim_probe_fill(16, 0, 16, None) == -1
    assert L.rlsim_probe_fill(16, (1 << 20) + 1, 16, None) == -1
    assert L.rlsim_probe_fill(1 << 40, 1, 16, None) == -1              # grid of 2^32 workgroups
    assert L.rlsim_probe_fill(16, 1, None, None) == -1
    out = probe.Dispatch()
    assert L.rlsim_probe_dispatch(0, 0, 1, 1, 256, out) == -1
    assert L.rlsim_probe_dispatch(1, 0, 0, 1, 256, out) == -1
    assert L.rlsim_probe_dispatch(1, 0, 1, 1, 0, out) == -1
    assert L.rlsim_probe_dispatch(1, 0, 1, 1, 256, None) == -1
    assert L.rlsim_probe_fill(16, 1, 20, None) == -1                  # misaligned dst


def test_probe_issues_each_steps_stores_back_to_back(tmp_path):
    """The store probe's time is the layout's ceiling only in its fastest
    order: the seven stores of a step with nothing between them, byte planes
    first.  The compiler chooses the schedule, so the built assembly is read."""
    from paper_2207_07736_amd import build
    out = build.asm(str(tmp_path / "probe.s"), build.PROBE_SRCS[0])
    text = open(out).read()
    name = next(l.split(":")[0] for l in text.splitlines() if l.startswith("_ZN9rlsim_dev13k_store_probe"))
    body = text[text.index(name + ":"):]
    body = body[:body.index("s_endpgm")].splitlines()
    code = [l.split()[0] for l in body if l.strip() and not l.strip().startswith((";", "."))]
    stores = [i for i, op in enumerate(code) if op.startswith("global_store")]
    assert len(stores) == 7 and stores[-1] - stores[0] == 6, [code[i] for i in range(stores[0], stores[-1] + 1)]
    assert [code[i] for i in stores] == ["global_store_byte"] * 2 + ["global_store_dword"] * 5


def test_create_rejects_every_invalid_cfg_drawn():
    """Seeded draws of configurations that break one rule each (a non-finite
    constant, a non-positive mass, length or step, an inverted range, an
    unknown flag, a zero compute factor): rlsim_create returns EINVAL with a
    message and touches no device."""
    import math
    import paper_2207_07736_amd as p
    rng = np.random.Generator(np.random.PCG64(77))
    floats = ["gravity", "masscart", "masspole", "half_length", "force_mag", "tau", "x_threshold",
              "theta_threshold_rad", "reset_low", "reset_high", "pad_a_low", "pad_a_high", "pad_b_low", "pad_b_high"]
    for _ in range(300):
        c = p.rlsim_cfg_default()
        kind = int(rng.integers(0, 6))
        if kind == 0:
            setattr(c, floats[int(rng.integers(len(floats)))], float(rng.choice([math.nan, math.inf, -math.inf])))
        elif kind == 1:
            setattr(c, str(rng.choice(["masscart", "masspole", "half_length", "tau"])), -float(rng.uniform(0, 5)))
        elif kind == 2:
            lo, hi = str(rng.choice(["reset", "pad_a", "pad_b"])) + "_low", None
            hi = lo.replace("_low", "_high")
            setattr(c, lo, getattr(c, hi) + float(rng.uniform(0.01, 3)))
        elif kind == 3:
            c.flags = int(rng.integers(2, 2**32))
        elif kind == 4:
            c.compute_factor = 0
        else:
            c.masscart = 0.0
        h = ctypes.c_void_p()
        rc = p.lib.rlsim_create(16, 4, ctypes.byref(c), ctypes.byref(h))
        assert rc == p.RLSIM_EINVAL and not h.value, (kind, rc)
        assert p.rlsim_last_error(None).startswith("rlsim_create: cfg")


@pytest.mark.parametrize("env0,n", [(1, 16), (255, 16), (2**32 - 256, 512), (2**32 - 2**20, 2**20 + 1)])
def test_create_rejects_bad_env0(env0, n):
    """Global env ids are 32-bit and blocks of 256 envs: env0 must be a multiple
    of 256 and env0 + n_envs <= 2^32, checked before any device call."""
    import paper_2207_07736_amd as p
    c = p.rlsim_cfg_default()
    assert c.env0 == 0
    c.env0 = env0
    h = ctypes.c_void_p()
    assert p.lib.rlsim_create(n, 4, ctypes.byref(c), ctypes.byref(h)) == p.RLSIM_EINVAL and not h.value
    assert "env0" in p.rlsim_last_error(None)


@pytest.mark.parametrize("model,links,words", [(2, 0, 4), (1, 0, 2), (1, 5, 12), (1, 2, 4), (1, 2, 7), (1, 1, 5)])
def test_create_rejects_bad_model_or_chain_shape(model, links, words):
    """An unknown model, a chain with n_links outside [1, 4], or a chain whose
    state_words is not 2 n_links + 2 (no padding words) is EINVAL."""
    import paper_2207_07736_amd as p
    c = p.rlsim_cfg_default()
    assert c.model == p.RLSIM_MODEL_CARTPOLE and c.n_links == 0
    c.model, c.n_links = model, links
    h = ctypes.c_void_p()
    assert p.lib.rlsim_create(64, words, ctypes.byref(c), ctypes.byref(h)) == p.RLSIM_EINVAL and not h.value
    assert p.rlsim_last_error(None).startswith("rlsim_create")


def test_trajectory_rows_carry_their_shape():
    """Rows cut from a Trajectory know the call they fit; statistics-only
    records check their buffer's size.  (Simulator.step compares them with
    the call before any launch; tests/test_gpu_parity.py runs that.)"""
    from paper_2207_07736_amd import rlsim
    torch = pytest.importorskip("torch")
    tr = rlsim.Trajectory(10, 300, device="cpu", S=6)
    r = tr.rows(2, 5)
    assert (r.K, r.n, r.S) == (5, 300, 6)
    assert r.obs == tr.obs[2:7].data_ptr()
    r.logp = None
    with pytest.raises(ValueError):
        r.obs = 1234
    for k0, k in ((0, 0), (8, 3), (-1, 2)):
        with pytest.raises(ValueError):
            tr.rows(k0, k)
    with pytest.raises(ValueError):
        rlsim.stats_only(torch.zeros((1, 4), dtype=torch.int32), 300)
    assert rlsim.stats_only(torch.zeros((2, 4), dtype=torch.int32), 300).K is None
