"""Host-side checks that need no GPU: the C-ABI library exports what include/pw.h declares, the
binding covers it, the product path refuses to run without a GPU, and host-only arithmetic."""
import ctypes as C
import os
import re

import pytest

from paper_2203_12533_amd import binding as pwb
from paper_2203_12533_amd import inputs as I

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_in_header():
    text = open(os.path.join(ROOT, "include", "pw.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(pw_[a-z0-9_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    names = _declared_in_header()
    assert len(names) >= 40
    lib = C.CDLL(pwb.LIB_PATH)
    for n in names:
        assert hasattr(lib, n), f"libpw.so lacks {n}"


def test_binding_covers_the_header():
    assert sorted(pwb.DECLARED_SYMBOLS) == _declared_in_header()
    pwb.lib()      # sets every signature; raises if one is missing


def test_struct_layouts_match_the_header(tmp_path):
    """The ctypes mirrors against the C compiler's view of include/pw.h: size of every struct that crosses the
    boundary, and the offset of each struct's last field."""
    structs = [("pw_tensor_spec", pwb.TensorSpec, "dims"), ("pw_fn_desc", pwb.FnDesc, "params_bytes"),
               ("pw_lm_config", pwb.LMConfigC, "fused_head_loss"), ("pw_stage_params", pwb.StageParams, "microbatch"),
               ("pw_gemm_args", pwb.GemmArgs, "xent"), ("pw_adam_epilogue", pwb.AdamEpilogue, "t"),
               ("pw_xent_epilogue", pwb.XentEpilogue, "inv_n"), ("pw_mha_args", pwb.MhaArgs, "causal"), ("pw_encdec_config", pwb.EncDecConfigC, "fused_update"), ("pw_node", pwb.Node, "in"),
               ("pw_sched_slice", pwb.SchedSlice, "end_ms"), ("pw_gemm_shape_row", pwb.GemmShapeRow, "total_flops")]
    src = tmp_path / "sizes.c"
    lines = ['#include <stdio.h>', '#include <stddef.h>', '#include "pw.h"', 'int main(void) {']
    for cname, _, last in structs:
        lines.append(f'  printf("%zu %zu\\n", sizeof({cname}), offsetof({cname}, {last}));')
    lines += ['  return 0;', '}']
    src.write_text("\n".join(lines))
    exe = tmp_path / "sizes"
    import subprocess
    subprocess.check_call(["gcc", "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe)])
    out = subprocess.check_output([str(exe)], text=True).split()
    for k, (cname, ct, last) in enumerate(structs):
        size, off = int(out[2 * k]), int(out[2 * k + 1])
        assert C.sizeof(ct) == size, cname
        py_last = ct._fields_[-1][0]
        assert getattr(ct, py_last).offset == off, (cname, last)


def test_environment_variables_of_the_library_carry_its_prefix():
    """A switch without the prefix takes another program's variable for its own."""
    csrc, read = os.path.join(os.path.dirname(pwb.LIB_PATH), "csrc"), set()
    for name in os.listdir(csrc):
        with open(os.path.join(csrc, name)) as f:
            read |= set(re.findall(r"getenv\(\s*([^)]*?)\s*\)", f.read()))
    assert read and all(re.fullmatch(r'"PW_[A-Z0-9_]+"', v) for v in read), read


def test_no_gpu_means_a_loud_failure_not_a_fallback():
    import torch
    if torch.cuda.is_available():
        pytest.skip("a GPU is present")
    with pytest.raises(pwb.PwError) as e:
        pwb.Context(0)
    assert e.value.status in (pwb.PW_ERR_DEVICE, pwb.PW_ERR_UNSUPPORTED)


def test_null_arguments_are_rejected_without_a_context():
    lib = pwb.lib()
    assert lib.pw_ctx_create(0, None, None) == pwb.PW_ERR_INVALID
    assert lib.pw_ctx_destroy(None) == pwb.PW_ERR_INVALID
    assert lib.pw_compile_fn(None, None, None) == pwb.PW_ERR_INVALID
    assert lib.pw_run_fn(None, 0, None, 0, None, 0) == pwb.PW_ERR_INVALID
    assert lib.pw_await(None, 0, None, 0) == pwb.PW_ERR_INVALID
    assert lib.pw_model_param_count(None) == -1


def test_model_flops_of_the_measured_workloads():
    # 6 N (L 12 d^2 + d V) + 6 B T^2 d L, the convention the throughput is priced with
    c3 = I.workload("cfg3")
    want = 6 * 8192 * (12 * 12 * 2048 ** 2 + 2048 * 32768) + 6 * 8 * 1024 ** 2 * 2048 * 12
    assert pwb.step_flops(c3) == pytest.approx(want, rel=1e-12)
    assert pwb.step_flops(c3) == pytest.approx(34.2e12, rel=5e-3)
    assert pwb.step_flops(I.workload("cfg1")) == pytest.approx(5.64e9 + 0.20e9, rel=1e-2)
    assert pwb.step_flops(I.workload("cfg4")) == pytest.approx(82.5e12, rel=5e-3)
    assert pwb.step_flops(I.workload("cfg5")) == pytest.approx(47.0e12, rel=5e-3)


def test_generator_is_counter_based_and_reproducible():
    import numpy as np
    a = I.normal(5, 9, 1000)
    b = I.normal(5, 9, 2000)
    assert np.array_equal(a, b[:1000])                      # a prefix does not depend on the length drawn
    assert not np.array_equal(a, I.normal(6, 9, 1000))
    t = I.lm_tokens(I.workload("cfg1"))
    assert t.shape == (4, 129) and t.min() >= 0 and t.max() < 1024
    w = I.lm_params(I.workload("cfg3").with_(n_layer=1, vocab=64, seq=8))
    assert np.array_equal(I.round_to_bf16(w["l0.wo"]), w["l0.wo"])   # bf16 workloads start bf16-representable
    x = np.array([1.0, 1.00390625, 1.01171875, -3.0e-41], dtype=np.float32)
    r = I.round_to_bf16(x)
    assert r[0] == 1.0 and r[1] == 1.0 and r[2] == np.float32(1.015625)   # ties to even, both directions


def test_bench_refuses_more_than_one_gpu_and_its_sampler_survives_missing_sysfs(tmp_path):
    """bench.py --gpus 2 exits with a message (one GPU only); the clock / power sampler of the timed region is a
    host thread reading sysfs and must return a plain dict whether or not the files exist."""
    import importlib.util
    import subprocess
    import sys
    root = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..")
    r = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"], capture_output=True, text=True)
    assert r.returncode == 2 and "ONE GPU" in r.stderr
    spec = importlib.util.spec_from_file_location("pw_bench", os.path.join(root, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    s = bench.ClockPowerSampler()
    s.sclk, s.power, s.cap = [str(tmp_path / "absent")], [str(tmp_path / "absent")], [str(tmp_path / "absent")]
    s.start()
    assert s.stop() == {}
    (tmp_path / "sclk").write_text("0: 500Mhz\n1: 2100Mhz *\n2: 2400Mhz\n")
    (tmp_path / "power").write_text("1350000000\n")
    (tmp_path / "cap").write_text("1400000000\n")
    s = bench.ClockPowerSampler()
    s.sclk, s.power, s.cap = [str(tmp_path / "sclk")], [str(tmp_path / "power")], [str(tmp_path / "cap")]
    s.start()
    import time
    time.sleep(0.12)
    note = s.stop()
    assert note["sclk_mhz_during_timed_steps"]["mean"] == 2100 and note["board_power_w_during_timed_steps"]["max"] == 1350
    assert note["board_power_cap_w"] == 1400


def test_device_version_of_the_input_generator_draws_the_same_numbers():
    """bench.py and the full-size GPU tests draw the 0.7 G weights of the measured workload with inputs.normal_torch;
    on the CPU it must reproduce inputs.normal: identical random bits, values equal after the rounding to float32 up
    to rare last-place differences of the float64 logarithm / cosine, and equal distribution parameters."""
    import numpy as np
    import torch
    n = 200_000
    for seed, tid, std in ((1234, 77, 0.02), (5, I._tid("l3.w1"), 1.0)):
        a = I.normal(seed, tid, n, std)
        b = I.normal_torch(seed, tid, n, std, "cpu").numpy()
        assert (a != b).mean() < 1e-4
        assert np.abs(a - b).max() <= np.abs(a).max() * 2.0 ** -22
    cfg = I.workload("cfg3").with_(n_layer=1, vocab=512, seq=16)
    ref = I.lm_params(cfg)
    for name, shape, kind in I.param_shapes(cfg):
        got = I.param_torch(cfg, name, shape, kind, "cpu").numpy().reshape(shape)
        assert (got != ref[name]).mean() < 1e-4, name
        assert np.array_equal(I.round_to_bf16(got), got)          # bf16-representable
