"""Which kernels the library launches, without a GPU: in a process of its own whose HIP runtime is tests/hip_recorder.c."""
import os
import subprocess
import sys

import pytest

from util import PATCH_SHARES

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

pytestmark = pytest.mark.skipif(not os.path.exists(os.path.join(ROOT, "paper_2110_15238_amd", "libbolt.so")),
                                reason="libbolt.so not built (run __graft_entry__.build())")

PRELUDE = """
import ctypes as C, sys
sys.path.insert(0, %r)
import paper_2110_15238_amd as b
lib, rec = b.binding.raw(), C.CDLL(%r)
rec.recorder_launches.restype = C.c_char_p
P = 0x10000  # stands for every device pointer

def cost(name, ms, repeated=None):
    rec.recorder_cost(name.encode(), C.c_float(ms), C.c_float(ms if repeated is None else repeated))

def conv(d, cfg=None, res=False):  # status and kernels of one call
    c = None if cfg is None else C.byref(b.BoltConfig.from_dict(cfg))
    if res: s = lib.bolt_conv2d_fprop_nhwc_residual(C.byref(d), P, P, P, P, 1.0, P, c, None, 0, None)
    else: s = lib.bolt_conv2d_fprop_nhwc(C.byref(d), P, P, P, P, c, None, 0, None)
    return s, rec.recorder_launches().decode().split()
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("recorder") / "hip_recorder.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "hip_recorder.c")], check=True)

    def go(code):
        env = dict(os.environ, LD_PRELOAD=":".join([so] + os.environ.get("LD_PRELOAD", "").split(":")).rstrip(":"))
        r = subprocess.run([sys.executable, "-c", PRELUDE % (ROOT, so) + code], env=env, capture_output=True, text=True)
        assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
        return r.stdout

    return go


def test_a_remembered_pick_is_for_its_alpha_and_activation(run):
    """The pick rule takes conv_patch_kernel for alpha = 1 with ReLU or nothing: after such a call the same sizes with another alpha or
    activation run on another kernel, as they do alone, and the first call runs on it again."""
    run("""
d = lambda alpha, act: b.conv_desc(8, 56, 56, 64, 64, 3, 3, 1, 1, alpha=alpha, act=act)
for turn in range(2):
    for alpha, act, patch in ((1.0, "relu", True), (0.5, "relu", False), (1.0, "relu", True), (1.0, "gelu", False), (0.5, "none", False), (1.0, "none", True)):
        s, kernels = conv(d(alpha, act))
        assert s == 0 and len(kernels) == 1, (s, kernels)
        assert ("conv_patch_kernel" in kernels[0]) == patch, (turn, alpha, act, kernels)
""")


@pytest.mark.parametrize("shape", [(2, 56, 56, 64, 64), (2, 28, 28, 32, 40), (2, 28, 28, 128, 128), (2, 14, 14, 256, 256), (2, 7, 7, 512, 512)])
def test_every_instance_of_a_plain_3x3_takes_a_residual(run, shape):
    """A config that bolt_tune found for the plain op (any legal instance) is valid with a residual, on that instance; without a config
    the call keeps to the kernels whose cost with a residual the pick rule knows."""
    run("""
d, ids = b.conv_desc(%d, %d, %d, %d, %d, 3, 3, 1, 1), []
for kid in range(b.bolt_num_instances(b.OP_CONV2D)):
    if not b.bolt_instance_supports(b.OP_CONV2D, kid, d): continue
    plain, res = conv(d, dict(kernel_id=kid)), conv(d, dict(kernel_id=kid), True)
    assert plain[0] == 0 and res[0] == 0 and len(res[1]) == 1, (kid, plain, res)
    assert plain[1][0].split("Li")[0] == res[1][0].split("Li")[0], (plain, res)
    ids += [kid] * ("conv_slice" in plain[1][0] or "conv_patch" in plain[1][0])
assert ids
s, kernels = conv(d, res=True)
assert s == 0 and not any(k in kernels[0] for k in ("conv_slice", "conv_patch")), kernels
""" % shape)


def test_a_pair_or_3x3_tuned_with_relu_takes_any_activation_and_alpha(run):
    """Legality is a matter of sizes: every instance that runs a problem with ReLU and alpha = 1 runs it with the others, by its config;
    without one such a call stays off conv_patch_kernel, whose costs the pick rule knows for the plain form."""
    run("""
def pair(c0, c1, cfg=None):
    c = None if cfg is None else C.byref(b.BoltConfig.from_dict(cfg))
    return lib.bolt_b2b_conv(C.byref(c0), C.byref(c1), P, P, P, P, P, P, c, None, 0, None), rec.recorder_launches().decode().split()
others = (("gelu", 1.0), ("relu", 0.5), ("softplus", -1.0), ("hardswish", 1.0), ("none", 2.0))
d = lambda act="relu", alpha=1.0: b.conv_desc(8, 56, 56, 64, 64, 3, 3, 1, 1, alpha=alpha, act=act)
e = lambda act="relu", alpha=1.0: b.conv_desc(8, 56, 56, 64, 256, 1, 1, alpha=alpha, act=act)
ran = 0
for kid in range(b.bolt_num_instances(b.OP_CONV2D)):
    if b.bolt_instance_supports(b.OP_CONV2D, kid, d()):
        for o in others:
            assert conv(d(*o), dict(kernel_id=kid))[0] == 0, (kid, o)
            ran += 1
for kid in range(b.bolt_num_instances(b.OP_B2B_CONV)):
    if b.bolt_instance_supports(b.OP_B2B_CONV, kid, d(), e()):
        for o in others:
            assert pair(d(*o), e(), dict(kernel_id=kid))[0] == 0 and pair(d(), e(*o), dict(kernel_id=kid))[0] == 0, (kid, o)
            ran += 1
assert ran >= 30
for o in others:
    for s, kernels in (conv(d(*o)), pair(d(*o), e()), pair(d(), e(*o))):
        assert s == 0 and "conv_patch" not in kernels[0], (o, kernels)
assert "conv_patch" in conv(d())[1][0] and "conv_patch" in pair(d(), e())[1][0]
""")


def test_last_units_of_a_pair_are_shared_where_they_leave_waves_idle(run):
    """The sharing form of conv_patch_kernel, plain and general, is launched for pairs with a residual whose last round is at most half full, on
    every instance of the family; not without a residual, nor where whole rounds are left."""
    run("""
cases = %r
ran = set()
for (n, h, w, c, k0, r, stride, pad, k1), share in cases:
    c0 = b.conv_desc(n, h, w, c, k0, r, r, stride, pad)
    p, q = b.conv_out_hw(c0)
    plain = b.conv_desc(n, p, q, k0, k1, 1, 1)
    for kid in range(b.bolt_num_instances(b.OP_B2B_CONV)):
        if not b.bolt_instance_supports(b.OP_B2B_CONV, kid, c0, plain): continue
        cfg = C.byref(b.BoltConfig.from_dict(dict(kernel_id=kid)))
        for c1, general in ((plain, 0), (b.conv_desc(n, p, q, k0, k1, 1, 1, alpha=0.5), 1)):
            assert lib.bolt_b2b_conv(C.byref(c0), C.byref(c1), P, P, P, P, P, P, cfg, None, 0, None) == 0
            assert lib.bolt_b2b_conv_residual(C.byref(c0), C.byref(c1), P, P, P, P, P, P, 1.0, P, cfg, None, 0, None) == 0
            alone, skip = rec.recorder_launches().decode().split()
            if "conv_patch_kernel" not in alone: continue
            assert "ELb1ELb0ELb%%dELb0EEE" %% general in alone and "ELb1ELb1ELb%%dELb%%dEEE" %% (general, share > 1) in skip, (n, h, w, share, alone, skip)
            ran.add((share, general))
assert ran == {(s, g) for s in (1, 2, 3, 4) for g in (0, 1)}, ran
""" % (PATCH_SHARES,))


@pytest.mark.parametrize("after_itself", (0.014, 0.020, 0.026, 0.040))
def test_tuner_ranks_short_kernels_whatever_the_eviction_took(run, after_itself):
    """bolt_tune times a candidate together with a kernel that evicts the caches.  What that kernel takes by itself, back to back, is not what
    it takes between launches: if it takes longer, candidates of a few microseconds are still told apart."""
    run("""
cost("tune_evict", 0.020, %g); cost("conv_slice", 0.0030); cost("conv_halo", 0.0031); cost("", 0.0035)
d, best = b.conv_desc(8, 14, 14, 256, 256, 3, 3, 1, 1), b.BoltConfig()
ptrs = (C.c_void_p * 4)(P, P, P, P)
assert lib.bolt_tune(b.OP_CONV2D, C.byref(d), None, ptrs, None, 0, None, C.byref(best), None, None) == 0
rec.recorder_launches()
s, kernels = conv(d, dict(kernel_id=best.kernel_id))
assert s == 0 and "conv_slice" in kernels[0], kernels
""" % after_itself)
