"""A pipeline step that is refused leaves every block where it was, and the step can be repeated.  The library's host code runs here on
a runtime of host memory (host_runtime.cpp), in a process of its own: nothing is computed, but every launch is counted."""
import ctypes
import os
import subprocess
import sys
import types

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TICKS, REFUSED_AT = 9, 6  # (tick 6: every queue is full)
SCHEDULES = {"staggered": ((1, 1, 0), (4, 2, 0)), "forward-locked": ((0, 0, 0), (2, 1, 0))}


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    """The stand-in under the name and symbol versions the library asks for."""
    d = tmp_path_factory.mktemp("runtime")
    lib, ver = str(d / "libamdhip64.so.7"), str(d / "versions")
    with open(ver, "w") as f:
        f.write("hip_4.2 { global: *; };\nhip_4.3 { global: hipGraph*; hipStreamBeginCapture; hipStreamEndCapture; } hip_4.2;\n")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-pthread", "-Wl,-soname,libamdhip64.so.7",
                    "-Wl,--version-script," + ver, os.path.join(ROOT, "tests", "host_runtime.cpp"), "-o", lib], check=True)
    return lib


@pytest.mark.parametrize("fault", ["batch", "labels", "stream"])
@pytest.mark.parametrize("schedule", SCHEDULES)
def test_a_refused_step_can_be_repeated(runtime, schedule, fault):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), runtime, schedule, fault], capture_output=True, text=True,
                       timeout=100, cwd=ROOT)
    assert r.returncode == 0, r.stdout + r.stderr


def _run(rt, D, cfg, params, schedule, fault):
    """Launches of TICKS steps, the one at REFUSED_AT first with what `fault` names refused."""
    import numpy as np
    from workloads import flatten_params
    p, m = SCHEDULES[schedule]
    shapes, blocks = [tuple(cfg["input"])], []
    for k, layers in enumerate(cfg["blocks"]):
        desc, keep = D.make_block_desc(layers, shapes[-1], D.DSP_FP32, k, 3, m[k], p_prev=p[k - 1] if k else 0, needs_input_grad=k > 0)
        blocks.append(D.dsp_block_init(desc, flatten_params(layers, params[k])))
        shapes.append(D.dsp_block_output_shape(blocks[-1])[0])
    pl = D.dsp_pipeline_init(blocks, p, m, 0.1, 0.9, 0.0, TICKS)
    D.dsp_pipeline_set_graph_replay(pl, False)
    x, y, strange = ctypes.c_void_p(), ctypes.c_void_p(), np.zeros(int(np.prod(cfg["input"])), np.float32)
    rt.hipMalloc(ctypes.byref(x), ctypes.c_size_t(strange.nbytes))
    rt.hipMalloc(ctypes.byref(y), ctypes.c_size_t(4 * cfg["input"][0]))
    before, state = rt.host_runtime_launches(), lambda: ([D.dsp_block_query(b) for b in blocks], D.dsp_pipeline_ticks(pl), rt.host_runtime_launches())
    for t in range(TICKS):
        if fault and t == REFUSED_AT:
            was = state()
            bad = {"batch": (strange, y.value, 0), "labels": (x.value, strange, 0), "stream": (x.value, y.value, 0x7)}[fault]
            for _ in range(2):
                with pytest.raises(D.DSPError) as e:
                    D.dsp_pipeline_step(pl, bad[0], bad[1], stream=bad[2])
                assert "refused" in str(e.value)
                assert state() == was
        early = t > 0 and schedule == "staggered"
        if early:  # a mini-batch in device memory is copied while the launch threads are at work
            rt.host_runtime_await_launch(x)
        D.dsp_pipeline_step(pl, x.value, y.value, stream=0)
        assert not early or rt.host_runtime_saw_launch()
    launches = rt.host_runtime_launches() - before
    done = [D.dsp_block_query(b) for b in blocks]
    D.dsp_pipeline_destroy(pl)
    for b in blocks:
        D.dsp_block_destroy(b)
    return launches, done


def _main(path, schedule, fault):
    rt = ctypes.CDLL(path, mode=ctypes.RTLD_GLOBAL)  # before the library, which then takes it for the HIP runtime
    rt.host_runtime_launches.restype = ctypes.c_int64
    rt.host_runtime_caller()
    sys.path.insert(0, ROOT)
    sys.modules["torch"] = types.ModuleType("torch")  # the binding imports it for the sake of that runtime alone
    import numpy as np
    import paper_1909_02625_amd as D
    from workloads import get_config, make_params
    cfg = get_config("resnet20", batch=4, hw=8)
    rng = np.random.default_rng(0)
    params = [make_params(layers, rng) for layers in cfg["blocks"]]
    assert _run(rt, D, cfg, params, schedule, fault) == _run(rt, D, cfg, params, schedule, None)


if __name__ == "__main__":
    _main(*sys.argv[1:])
