"""Host-side checks that need no GPU: the library loads, exports every symbol the header declares,
sizes buffers consistently, and rejects bad specs before touching the device."""
import ctypes as C
import dataclasses
import os
import re

import pytest

import lp_inputs as LI
import paper_2012_03837_amd as lp
from paper_2012_03837_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def header_symbols():
    names = set()
    for fn in sorted(os.listdir(os.path.join(ROOT, "include"))):
        if fn.endswith(".h"):
            txt = open(os.path.join(ROOT, "include", fn)).read()
            txt = re.sub(r"/\*.*?\*/", "", txt, flags=re.S)
            names |= set(re.findall(r"\b(lpk?_[a-z0-9_]+)\s*\(", txt))
    return sorted(names)


def test_library_exports_every_declared_symbol():
    L = lp.lib()
    syms = header_symbols()
    assert "lp_init_blocks" in syms and "lp_local_step" in syms and "lp_eval_loss" in syms
    for s in syms:
        assert hasattr(L, s), s


@pytest.mark.parametrize("B,S,H,dh,backward,parts", [
    (1, 64, 2, 64, 1, 1), (1, 65, 2, 64, 1, 2), (1, 129, 2, 64, 1, 4), (2, 256, 8, 64, 1, 4), (2, 256, 9, 64, 1, 1),
    (4, 300, 8, 64, 1, 2), (4, 300, 8, 64, 0, 4), (4, 300, 8, 32, 1, 4), (2, 300, 8, 64, 1, 4), (3, 300, 7, 64, 1, 2),
    (2, 512, 8, 64, 1, 4), (2, 512, 10, 64, 1, 2), (2, 768, 8, 64, 1, 2), (1, 1024, 12, 64, 1, 4), (1, 1536, 8, 64, 1, 4), (1, 2048, 7, 64, 1, 2),
    (4, 512, 11, 64, 1, 2), (4, 512, 12, 64, 1, 1), (4, 512, 8, 64, 0, 4), (3, 512, 11, 64, 0, 2), (8, 512, 8, 16, 0, 2), (13, 512, 5, 16, 0, 1),
    (1, 512, 8, 48, 0, 0), (0, 512, 8, 64, 0, 0)])
def test_attention_parts_follow_the_measurements(B, S, H, dh, backward, parts):
    """The rule at both sides of its limits.  Four parts of 64-wide heads' backward pass beyond them: 96 blocks of 300 positions
    15.9 us, 15.4 whole and 13.0 in two."""
    from paper_2012_03837_amd import kernels as K
    assert K.lpk_attention_parts(B, S, H, dh, backward) == parts


def test_query_sizes_all_configs():
    import numpy as np
    for name in LI.CONFIG_NAMES:
        cfg = LI.make_config(name)
        spec, keep = lp.make_spec(cfg)
        sz = lp.lp_query_sizes(spec)
        n_par = sum(int(np.prod(s)) for s in LI.param_shapes(cfg).values())
        per = 4 + (2 if cfg.dtype == "bf16" else 0)
        assert sz.param_bytes >= n_par * per
        assert sz.param_bytes < n_par * per * 1.01 + (1 << 20)
        n_state = {"sgd": 0, "sgdm": 1, "adam": 2}[cfg.opt.kind]
        assert sz.state_bytes >= n_par * 4 * n_state
        assert sz.work_bytes > n_par * 4
        assert sz.param_bytes % 256 == 0 and sz.state_bytes % 256 == 0 and sz.work_bytes % 256 == 0
        assert sz.work_bytes < 64 << 30


def _status(fn):
    with pytest.raises(lp.LpError) as e:
        fn()
    return e.value.status, str(e.value)


def test_bad_specs_are_rejected_on_the_host():
    cfg = LI.make_config("cfg3_small")

    def q(c, **kw):
        spec, keep = lp.make_spec(c, **kw)
        return lambda: lp.lp_query_sizes(spec)

    bad_window = dataclasses.replace(cfg, heads=(dataclasses.replace(cfg.heads[0], window=0),) + cfg.heads[1:])
    assert _status(q(bad_window))[0] == B.LP_EINVAL
    unordered = dataclasses.replace(cfg, heads=cfg.heads[::-1])
    assert _status(q(unordered))[0] == B.LP_EINVAL
    bad_heads = dataclasses.replace(cfg, layers=tuple(dataclasses.replace(l, n_heads=3) for l in cfg.layers))
    assert _status(q(bad_heads))[0] == B.LP_ESHAPE
    assert _status(q(cfg, max_batch=0))[0] == B.LP_ESHAPE
    wrong_in = dataclasses.replace(cfg, heads=(dataclasses.replace(cfg.heads[0], in_dim=64),) + cfg.heads[1:])
    st, msg = _status(q(wrong_in))
    assert st == B.LP_ESHAPE and "head 1" in msg
    mlp = LI.make_config("cfg1")
    mixed = dataclasses.replace(mlp, layers=mlp.layers[:1] + cfg.layers[:1])
    assert _status(q(mixed))[0] in (B.LP_EUNSUPPORTED, B.LP_ESHAPE)
    # null spec
    assert lp.lib().lp_query_sizes(None, None) == B.LP_EINVAL


def test_init_rejects_null_and_misaligned_buffers_before_any_device_call():
    cfg = LI.make_config("cfg1")
    spec, keep = lp.make_spec(cfg)
    assert _status(lambda: lp.lp_init_blocks(spec, 0, 0, 0))[0] == B.LP_EINVAL
    assert _status(lambda: lp.lp_init_blocks(spec, 0x1000 + 8, 0x2000, 0x3000))[0] == B.LP_EALIGN
    ctx = C.c_void_p(123)
    bufs = B.lp_buffers(0, 0, 0)
    st = lp.lib().lp_init_blocks(C.byref(spec), C.byref(bufs), None, C.byref(ctx))
    assert st == B.LP_EINVAL and ctx.value is None


def test_null_context_calls_fail_cleanly():
    L = lp.lib()
    assert L.lp_local_step(None, None, None, 1, None) == B.LP_EINVAL
    assert L.lp_eval_loss(None, None, None, 1, None) == B.LP_EINVAL
    assert L.lp_get_tensor(None, b"L1.w1", None, 0) == B.LP_EINVAL
    assert L.lp_num_params(None) == 0
    assert L.lp_step_graph(None, 1) == B.LP_EINVAL
    assert L.lp_bn_running(None, 0.1, 0) == B.LP_EINVAL
    assert L.lp_overlap_steps(None, 1) == B.LP_EINVAL
    assert L.lp_join(None) == B.LP_EINVAL
    L.lp_destroy(None)


def test_bench_refuses_more_than_one_gpu():
    """Every box has one GPU: asking the bench for more ends with a message, before anything touches a device."""
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode != 0
    assert "--gpus must be 1" in r.stderr
    assert not r.stdout.strip()


def test_scratch_sets_of_a_residual_mlp():
    """bf16 with two streams or more: chains, a whole scratch set per stream, however many heads there are.  fp32: the blocks
    run in lockstep, a set per head, whatever the streams."""
    def work(dtype, ns):
        cfg = dataclasses.replace(LI.configs.mlp_config("t", n_layers=4), dtype=dtype)
        spec, keep = lp.make_spec(cfg, n_streams=ns)
        return lp.lp_query_sizes(spec).work_bytes

    def step(dtype, ns):
        return work(dtype, ns + 1) - work(dtype, ns)

    assert step("bf16", 2) == step("bf16", 7)
    assert step("f32", 2) < step("f32", 7)


def test_filter_gradient_without_output_pixels_returns_on_the_host():
    """A 3 x 3 filter on a 2 x 2 image without padding has no output: the call's host part divides by no output size.  In a
    process of its own without a device, where the launch behind it is an error code."""
    import subprocess
    import sys
    code = ("import ctypes as C\nfrom paper_2012_03837_amd.binding import lib\n"
            "print(lib().lpk_conv_bwd_weight(1, C.c_void_p(4096), C.c_void_p(8192), C.c_void_p(16384), 2, 2, 2, 8, 8, 3, 1, 0, 0, C.c_void_p(0)))")
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, env=dict(os.environ, HIP_VISIBLE_DEVICES="-1"), capture_output=True,
                       text=True, timeout=300)
    assert r.returncode == 0 and int(r.stdout.split()[-1]) != 0, (r.returncode, r.stderr)


def test_products_bound_by_their_output_choose_by_it():
    """The kernel that a short reduction over a large output takes (printed in front of the launch, which fails without a
    device): whole lines from 256-wide tiles where nothing is fused, one tile per block where something is (8192 x 16384 x 64:
    64 and 89 us, and 102 and 147 us with the 256 x 128 tiles), and 128 x 128 tiles where they make one full round."""
    import subprocess
    import sys
    code = ("import ctypes as C\nfrom paper_2012_03837_amd.binding import lib\n"
            "v, n = C.c_void_p, C.c_int64\n"
            "for M, N, K, bias in ((8192, 16384, 64, 0), (8192, 32000, 32, 0), (8192, 16384, 64, 4096), (528, 11648, 112, 0)):\n"
            "    lib().lpk_gemm(1, v(4096), n(K), 1, v(8192), n(K), 1, v(16384), n(N), 0, M, N, K, v(bias), 0, v(0), v(0), 0, n(0),\n"
            "                   v(0), n(0), 0, 0, v(0), C.c_size_t(0), v(0))\n")
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, env=dict(os.environ, HIP_VISIBLE_DEVICES="-1", LP_GEMM_TRACE="1"),
                       capture_output=True, text=True, timeout=300)
    took = re.findall(r"\(11\): (persistent, kind \d|tiles, shape \d)", r.stderr)
    assert r.returncode == 0 and len(took) == 4, r.stderr
    assert took[0] in ("persistent, kind 1", "persistent, kind 3") and took[1] == "persistent, kind 1", took
    assert took[2].startswith("tiles") and took[3] == "tiles, shape 2", took
