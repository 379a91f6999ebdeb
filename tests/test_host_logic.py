"""CPU-only checks of the C-ABI library: it loads, exports what include/bolt.h declares, and its
descriptor validation returns the documented status for each kind of bad input (no kernel runs)."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2110_15238_amd", "libbolt.so")

pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libbolt.so not built (run __graft_entry__.build())")

OK, INVALID, UNSUPPORTED, ALIGNMENT, WORKSPACE, LAUNCH, ILLEGAL = range(7)


@pytest.fixture(scope="module")
def bolt():
    import paper_2110_15238_amd as b
    return b


def test_library_exports_every_declared_symbol():
    header = open(os.path.join(ROOT, "include", "bolt.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(bolt_[a-z0-9_]+)\s*\(", header))
    assert {"bolt_gemm_epilogue", "bolt_conv2d_fprop_nhwc", "bolt_b2b_gemm", "bolt_b2b_conv", "bolt_tune"} <= declared
    lib = ctypes.CDLL(LIB)
    for name in sorted(declared):
        assert hasattr(lib, name), name


def test_binding_lists_the_same_symbols(bolt):
    header = re.sub(r"/\*.*?\*/", "", open(os.path.join(ROOT, "include", "bolt.h")).read(), flags=re.S)
    declared = set(re.findall(r"\b(bolt_[a-z0-9_]+)\s*\(", header))
    assert declared == set(bolt.binding.EXPORTED)
    for name in declared:
        assert hasattr(bolt, name), name


def test_struct_layouts_match_header(bolt):
    assert ctypes.sizeof(bolt.BoltConfig) == 44
    assert ctypes.sizeof(bolt.GemmDesc) == 40
    assert ctypes.sizeof(bolt.ConvDesc) == 64


def test_instance_tables(bolt):
    for op in (bolt.OP_GEMM, bolt.OP_CONV2D, bolt.OP_B2B_GEMM, bolt.OP_B2B_CONV):
        n = bolt.bolt_num_instances(op)
        assert 10 <= n <= 256  # tens to a couple of hundred instances per op
        for i in range(n):
            c = bolt.bolt_instance_config(op, i).as_dict()
            assert c["kernel_id"] == i and c["tile_m"] % 32 == 0 and c["tile_n"] % 32 == 0
            assert c["waves_m"] * c["waves_n"] in (2, 4, 8)
    with pytest.raises(bolt.BoltError):
        bolt.bolt_instance_config(bolt.OP_GEMM, 10 ** 6)


def test_gemm_validation(bolt):
    G, chk = bolt.gemm_desc, bolt.bolt_check
    assert chk(bolt.OP_GEMM, G(256, 256, 256)) == OK
    assert chk(bolt.OP_GEMM, G(1, 8, 8)) == OK
    assert chk(bolt.OP_GEMM, G(0, 8, 8)) == INVALID
    assert chk(bolt.OP_GEMM, G(8, 8, -8)) == INVALID
    assert chk(bolt.OP_GEMM, G(256, 250, 256)) == ALIGNMENT        # N not a multiple of 8
    assert chk(bolt.OP_GEMM, G(256, 256, 100)) == ALIGNMENT        # K not a multiple of 8
    assert chk(bolt.OP_GEMM, G(256, 256, 256, lda=260)) == ALIGNMENT
    assert chk(bolt.OP_GEMM, G(256, 256, 256, lda=128)) == INVALID  # lda < K
    assert chk(bolt.OP_GEMM, G(256, 256, 256, ldd=8)) == INVALID
    d = G(256, 256, 256)
    d.act = 17
    assert chk(bolt.OP_GEMM, d) == INVALID
    d = G(256, 256, 256)
    d.b_layout = 5
    assert chk(bolt.OP_GEMM, d) == INVALID
    assert chk(bolt.OP_GEMM, None) == INVALID
    assert chk(bolt.OP_GEMM, G(64, 64, 64), None, {"kernel_id": 9999}) == INVALID
    assert chk(bolt.OP_GEMM, G(64, 64, 64), None, {"kernel_id": -1, "split_k": 1000}) == INVALID
    # an NK-layout instance cannot run a KN-layout problem
    n = bolt.bolt_num_instances(bolt.OP_GEMM)
    kn = [i for i in range(n) if bolt.bolt_instance_supports(bolt.OP_GEMM, i, G(512, 512, 512))]
    nk = [i for i in range(n) if bolt.bolt_instance_supports(bolt.OP_GEMM, i, G(512, 512, 512, b_layout=bolt.LAYOUT_NK))]
    assert kn and nk and not set(kn) & set(nk)
    assert chk(bolt.OP_GEMM, G(512, 512, 512), None, {"kernel_id": nk[0]}) == UNSUPPORTED
    # the direct-to-LDS instances for row-major weights address the whole weight matrix with 32-bit byte offsets:
    # from 2 GiB on only the register-staged instances remain
    sup = lambda K: {i for i in range(n) if bolt.bolt_instance_supports(bolt.OP_GEMM, i, G(512, 2048, K))}
    below, at = sup((1 << 19) - 8), sup(1 << 19)
    assert at and at < below
    assert all(bolt.bolt_instance_config(bolt.OP_GEMM, i).stages == 2 for i in at)
    assert chk(bolt.OP_GEMM, G(512, 2048, 1 << 19), None, {"kernel_id": max(below)}) == UNSUPPORTED


def test_conv_validation(bolt):
    Cd, chk = bolt.conv_desc, bolt.bolt_check
    assert chk(bolt.OP_CONV2D, Cd(32, 56, 56, 64, 64, 3, 3, 1, 1)) == OK
    # first layers: C <= 4 of either parity runs unpadded, from NHWC or NCHW, on the first-layer instances only
    stem = Cd(32, 224, 224, 3, 64, 7, 7, 2, 3)
    stem_nchw = Cd(32, 224, 224, 3, 64, 7, 7, 2, 3, x_layout="nchw")
    n = bolt.bolt_num_instances(bolt.OP_CONV2D)
    for d in (stem, stem_nchw):
        assert chk(bolt.OP_CONV2D, d) == OK
        ids = [i for i in range(n) if bolt.bolt_instance_supports(bolt.OP_CONV2D, i, d)]
        assert ids and all(bolt.bolt_instance_config(bolt.OP_CONV2D, i).tile_k == 32 for i in ids)
        assert all(not bolt.bolt_instance_supports(bolt.OP_CONV2D, i, Cd(32, 224, 224, 8, 64, 7, 7, 2, 3)) for i in ids)
    assert chk(bolt.OP_CONV2D, Cd(32, 224, 224, 5, 64, 7, 7, 2, 3)) == ALIGNMENT   # an odd C > 4 must be padded
    assert chk(bolt.OP_CONV2D, Cd(32, 224, 224, 8, 64, 7, 7, 2, 3, x_layout="nchw")) == UNSUPPORTED  # NCHW: C <= 4 only
    assert chk(bolt.OP_CONV2D, Cd(2, 64, 64, 3, 64, 9, 9, 2, 4)) == UNSUPPORTED    # R * C > 24: no first-layer instance
    assert chk(bolt.OP_CONV2D, Cd(2, 64, 64, 3, 64, 3, 3, 3, 1)) == UNSUPPORTED    # stride_w > 2
    assert chk(bolt.OP_CONV2D, Cd(2, 64, 64, 4, 64, 3, 3, 2, 1)) == OK             # C = 4: these or the alignment-2 ones
    bad = Cd(2, 64, 64, 3, 64, 3, 3, 1, 1)
    bad.x_layout = 7
    assert chk(bolt.OP_CONV2D, bad) == INVALID
    bad = Cd(2, 64, 64, 8, 64, 3, 3, 1, 1)
    bad.y_layout = 2
    assert chk(bolt.OP_CONV2D, bad) == INVALID
    # last layers: an NCHW output runs on the instances that have that store (and the first-layer kernels), and only there
    last = Cd(32, 7, 7, 512, 2048, 1, 1, 1, 0, y_layout="nchw")
    plain = Cd(32, 7, 7, 512, 2048, 1, 1, 1, 0)
    a = {i for i in range(n) if bolt.bolt_instance_supports(bolt.OP_CONV2D, i, last)}
    b = {i for i in range(n) if bolt.bolt_instance_supports(bolt.OP_CONV2D, i, plain)}
    assert a and b and not (a & b) and chk(bolt.OP_CONV2D, last) == OK
    assert chk(bolt.OP_CONV2D, last, None, {"kernel_id": min(b)}) == UNSUPPORTED
    assert chk(bolt.OP_CONV2D, last, None, {"kernel_id": min(a), "split_k": 2}) == UNSUPPORTED   # the reduction kernel writes NHWC
    assert chk(bolt.OP_CONV2D, Cd(2, 64, 64, 3, 64, 7, 7, 2, 3, x_layout="nchw", y_layout="nchw")) == OK
    assert chk(bolt.OP_B2B_CONV, Cd(2, 16, 16, 64, 64, 3, 3, 1, 1), Cd(2, 16, 16, 64, 64, 1, 1, 1, 0, y_layout="nchw")) == UNSUPPORTED
    assert chk(bolt.OP_B2B_CONV, Cd(2, 64, 64, 3, 64, 3, 3, 1, 1), Cd(2, 64, 64, 64, 64, 1, 1, 1, 0)) == ALIGNMENT
    assert chk(bolt.OP_CONV2D, Cd(32, 224, 224, 8, 64, 7, 7, 2, 3)) == OK
    # an even C that is not a multiple of 8: legal, and only the alignment-2 instances take it
    d46 = Cd(32, 20, 26, 46, 32, 3, 3, 1, 1)
    assert chk(bolt.OP_CONV2D, d46) == OK
    n = bolt.bolt_num_instances(bolt.OP_CONV2D)
    a2 = [i for i in range(n) if bolt.bolt_instance_supports(bolt.OP_CONV2D, i, d46)]
    a8 = [i for i in range(n) if bolt.bolt_instance_supports(bolt.OP_CONV2D, i, Cd(32, 20, 26, 48, 32, 3, 3, 1, 1))]
    assert len(a2) >= 3 and a8 and not set(a2) & set(a8)
    assert chk(bolt.OP_CONV2D, d46, None, {"kernel_id": a8[0]}) == UNSUPPORTED
    assert chk(bolt.OP_B2B_CONV, d46, Cd(32, 20, 26, 32, 64, 1, 1, 1, 0)) == ALIGNMENT  # fused kernels need C % 8 == 0
    assert chk(bolt.OP_CONV2D, Cd(1, 8, 8, 8, 12, 3, 3, 1, 1)) == ALIGNMENT
    assert chk(bolt.OP_CONV2D, Cd(1, 2, 2, 8, 8, 3, 3, 1, 0)) == INVALID            # filter larger than image
    assert chk(bolt.OP_CONV2D, Cd(1, 8, 8, 8, 8, 3, 3, 0, 1)) == INVALID            # stride 0
    assert chk(bolt.OP_CONV2D, Cd(1, 8, 8, 8, 8, 3, 3, 1, -1)) == INVALID
    assert chk(bolt.OP_CONV2D, Cd(4096, 1024, 1024, 8, 8, 3, 3, 1, 1)) == UNSUPPORTED  # 32-bit offsets
    assert bolt.conv_out_hw(Cd(1, 224, 224, 8, 64, 7, 7, 2, 3)) == (112, 112)


def test_first_layer_limits(bolt):
    """bolt.h's limits of the first layers (R * C <= 24, S <= 8, stride_w <= 2): what lies within runs in both layouts, and
    the strip kernels, which could run more, do not widen them.  4 channels from NHWC to NHWC have the alignment-2 kernels."""
    Cd = lambda c, r, s, sw, xl, yl="nhwc": bolt.bolt_check(bolt.OP_CONV2D, bolt.conv_desc(2, 40, 48, c, 64, r, s, (1, sw), 1, x_layout=xl, y_layout=yl))
    for c, r, s in ((3, 8, 8), (4, 6, 8), (1, 24, 8), (2, 12, 8), (3, 7, 7), (3, 1, 1)):
        for sw in (1, 2):
            for xl in ("nhwc", "nchw"):
                assert Cd(c, r, s, sw, xl) == OK and Cd(c, r, s, sw, xl, "nchw") == OK, (c, r, s, sw, xl)
    for c, r, s in ((4, 7, 7), (3, 9, 5), (3, 11, 2), (3, 9, 6)):  # within the strip kernels' 28 fragments
        assert Cd(c, r, s, 2, "nchw") == UNSUPPORTED and Cd(c, r, s, 2, "nhwc", "nchw") == UNSUPPORTED, (c, r, s)
        assert Cd(c, r, s, 2, "nhwc") == (OK if c == 4 else UNSUPPORTED), (c, r, s)
    assert Cd(4, 1, 15, 1, "nhwc") == OK


def test_b2b_fusion_legality(bolt):
    G, Cd, chk = bolt.gemm_desc, bolt.conv_desc, bolt.bolt_check
    assert chk(bolt.OP_B2B_GEMM, G(16384, 64, 256), G(16384, 128, 64)) == OK
    assert chk(bolt.OP_B2B_GEMM, G(16384, 64, 256), G(16000, 128, 64)) == ILLEGAL    # M must stay the same
    assert chk(bolt.OP_B2B_GEMM, G(16384, 64, 256), G(16384, 128, 72)) == ILLEGAL    # K1 must equal N0
    assert chk(bolt.OP_B2B_GEMM, G(16384, 64, 256), None) == INVALID
    assert chk(bolt.OP_B2B_GEMM, G(16384, 512, 256), G(16384, 128, 512)) == UNSUPPORTED  # no tile spans N0 = 512
    assert chk(bolt.OP_B2B_GEMM, G(16384, 128, 8192), G(16384, 64, 128)) == OK  # a W0 beyond LDS streams (multi-stage kernel)
    # row-major weights are addressed with 32-bit byte offsets: K0 * ldb * 2 must stay below 2 GiB
    assert chk(bolt.OP_B2B_GEMM, G(4096, 32, 1024, ldb=(1 << 20) - 8), G(4096, 32, 32)) == OK
    assert chk(bolt.OP_B2B_GEMM, G(4096, 32, 1024, ldb=1 << 20), G(4096, 32, 32)) == UNSUPPORTED
    c0 = Cd(32, 56, 56, 64, 64, 3, 3, 1, 1)
    assert chk(bolt.OP_B2B_CONV, c0, Cd(32, 56, 56, 64, 256, 1, 1, 1, 0)) == OK
    assert chk(bolt.OP_B2B_CONV, c0, Cd(32, 56, 56, 64, 256, 3, 3, 1, 1)) == ILLEGAL   # 2nd conv must be 1x1
    assert chk(bolt.OP_B2B_CONV, c0, Cd(32, 56, 56, 64, 256, 1, 1, 2, 0)) == ILLEGAL   # ... stride 1
    assert chk(bolt.OP_B2B_CONV, c0, Cd(32, 56, 56, 64, 256, 1, 1, 1, 1)) == ILLEGAL   # ... no padding
    assert chk(bolt.OP_B2B_CONV, c0, Cd(32, 56, 56, 128, 256, 1, 1, 1, 0)) == ILLEGAL  # C1 must equal K0
    assert chk(bolt.OP_B2B_CONV, c0, Cd(32, 28, 28, 64, 256, 1, 1, 1, 0)) == ILLEGAL   # extent must match
    c0s = Cd(32, 56, 56, 64, 64, 3, 3, 2, 1)
    assert chk(bolt.OP_B2B_CONV, c0s, Cd(32, 28, 28, 64, 64, 1, 1, 1, 0)) == OK
    # no compiled pair of widths is within 2x of (128, 16): the padding rule gives way rather than refuse the pair
    assert chk(bolt.OP_B2B_CONV, Cd(2, 12, 12, 64, 128, 3, 3, 1, 1), Cd(2, 12, 12, 128, 16, 1, 1, 1, 0)) == OK
    assert chk(bolt.OP_B2B_CONV, Cd(2, 12, 12, 64, 128, 3, 3, 1, 1), Cd(2, 12, 12, 128, 256, 1, 1, 1, 0)) == UNSUPPORTED  # no tile spans it


def test_fused_pair_residual_instance_sets(bolt):
    # the residual ops index the same instance tables; only the instances with that epilogue support them
    G, Cd = bolt.gemm_desc, bolt.conv_desc
    nk = bolt.LAYOUT_NK
    g0, g1 = G(16384, 64, 256, b_layout=nk), G(16384, 128, 64, b_layout=nk)
    c0, c1 = Cd(32, 56, 56, 64, 64, 3, 3, 1, 1), Cd(32, 56, 56, 64, 256, 1, 1, 1, 0)
    for plain, res, d0, d1 in ((bolt.OP_B2B_GEMM, bolt.OP_B2B_GEMM_RES, g0, g1), (bolt.OP_B2B_CONV, bolt.OP_B2B_CONV_RES, c0, c1)):
        n = bolt.bolt_num_instances(plain)
        assert bolt.bolt_num_instances(res) == n
        a = {i for i in range(n) if bolt.bolt_instance_supports(plain, i, d0, d1)}
        b = {i for i in range(n) if bolt.bolt_instance_supports(res, i, d0, d1)}
        assert b and b <= a
        assert bolt.bolt_check(res, d0, d1) == OK
        assert bolt.bolt_check(res, d0, d1, {"kernel_id": min(b)}) == OK
        assert bolt.bolt_instance_config(res, min(b)).as_dict() == bolt.bolt_instance_config(plain, min(b)).as_dict()
    # row-major weights: only the weights-resident kernels take them, and every one of them has the residual epilogue
    k0, k1 = G(16384, 64, 256), G(16384, 128, 64)
    n = bolt.bolt_num_instances(bolt.OP_B2B_GEMM)
    a = {i for i in range(n) if bolt.bolt_instance_supports(bolt.OP_B2B_GEMM, i, k0, k1)}
    b = {i for i in range(n) if bolt.bolt_instance_supports(bolt.OP_B2B_GEMM_RES, i, k0, k1)}
    assert b and b == a
    assert bolt.bolt_check(bolt.OP_B2B_GEMM_RES, k0, k1) == OK
    assert bolt.bolt_check(bolt.OP_B2B_GEMM_RES, g0, G(16000, 128, 64, b_layout=nk)) == ILLEGAL


def test_chain_legality(bolt):
    G, Cd, chk = bolt.gemm_desc, bolt.conv_desc, bolt.bolt_check_chain
    nk = bolt.LAYOUT_NK
    g = [G(4096, 64, 256, b_layout=nk), G(4096, 128, 64, b_layout=nk), G(4096, 64, 128, b_layout=nk)]
    assert chk(bolt.OP_GEMM_CHAIN3, g) == OK
    assert chk(bolt.OP_GEMM_CHAIN3, g[:2]) == UNSUPPORTED                                  # only three-op chains are compiled
    assert chk(bolt.OP_GEMM_CHAIN3, [g[0], g[1], G(4096, 64, 120, b_layout=nk)]) == ILLEGAL  # K2 must equal N1
    assert chk(bolt.OP_GEMM_CHAIN3, [g[0], g[1], G(4000, 64, 128, b_layout=nk)]) == ILLEGAL  # same M
    kn = [G(4096, 64, 256), G(4096, 128, 64), G(4096, 64, 128)]
    assert chk(bolt.OP_GEMM_CHAIN3, kn) == OK                                              # row-major weights: instances of their own
    assert chk(bolt.OP_GEMM_CHAIN3, [kn[0], kn[1], g[2]]) == UNSUPPORTED                   # ... but one layout per chain
    n3 = bolt.bolt_num_instances(bolt.OP_GEMM_CHAIN3)
    sup = lambda d: {i for i in range(n3) if bolt.bolt_chain_instance_supports(bolt.OP_GEMM_CHAIN3, i, d)}
    assert sup(kn) and sup(g) and not sup(kn) & sup(g)
    assert chk(bolt.OP_GEMM_CHAIN3, [g[0], g[1], G(4096, 512, 128, b_layout=nk)]) == UNSUPPORTED  # N2 beyond every bound
    assert chk(bolt.OP_GEMM, g) == INVALID
    assert chk(bolt.OP_GEMM_CHAIN3, g, {"kernel_id": 9999}) == INVALID
    c = [Cd(32, 56, 56, 64, 64, 3, 3, 1, 1), Cd(32, 56, 56, 64, 64, 1, 1, 1, 0), Cd(32, 56, 56, 64, 256, 1, 1, 1, 0)]
    assert chk(bolt.OP_CONV_CHAIN3, c) == OK
    assert chk(bolt.OP_CONV_CHAIN3, [c[0], c[1], Cd(32, 56, 56, 64, 256, 3, 3, 1, 1)]) == ILLEGAL   # later ops must be 1x1
    assert chk(bolt.OP_CONV_CHAIN3, [c[0], c[1], Cd(32, 28, 28, 64, 256, 1, 1, 1, 0)]) == ILLEGAL   # extent must carry over
    for op in (bolt.OP_GEMM_CHAIN3, bolt.OP_CONV_CHAIN3):
        n = bolt.bolt_num_instances(op)
        assert n >= 8
        descs = g if op == bolt.OP_GEMM_CHAIN3 else c
        ok = [i for i in range(n) if bolt.bolt_chain_instance_supports(op, i, descs)]
        assert ok and all(bolt.bolt_instance_config(op, i).as_dict()["tile_n"] >= descs[2].N if op == bolt.OP_GEMM_CHAIN3
                          else True for i in ok)


def test_a_configuration_is_not_bound_to_the_row_count(bolt):
    """An id that bolt_tune may return for one batch stays legal for every other: how many rows a kernel is worth using at
    is a matter of the pick rule and of the tuner's candidates."""
    G, Cd, rows = bolt.gemm_desc, bolt.conv_desc, (1, 32, 1000, 30000, 131072)
    sets = []
    for layout in (bolt.LAYOUT_KN, bolt.LAYOUT_NK):
        for n, k in ((1000, 2048), (64, 256)):
            sets.append([{i for i in range(bolt.bolt_num_instances(bolt.OP_GEMM))
                          if bolt.bolt_instance_supports(bolt.OP_GEMM, i, G(m, n, k, b_layout=layout))} for m in rows])
        for n0, n1, k in ((64, 32, 96), (64, 128, 128), (128, 64, 576)):
            sets.append([{i for i in range(bolt.bolt_num_instances(bolt.OP_B2B_GEMM)) if bolt.bolt_instance_supports(
                bolt.OP_B2B_GEMM, i, G(m, n0, k, b_layout=layout), G(m, n1, n0, b_layout=layout))} for m in rows])
        sets.append([{i for i in range(bolt.bolt_num_instances(bolt.OP_GEMM_CHAIN3)) if bolt.bolt_chain_instance_supports(
            bolt.OP_GEMM_CHAIN3, i, [G(m, 32, 96, b_layout=layout), G(m, 96, 32, b_layout=layout), G(m, 32, 96, b_layout=layout)])}
            for m in rows])
    for h, c, r, stride in ((14, 256, 3, 1), (56, 64, 1, 2), (12, 46, 3, 1), (32, 3, 3, 2)):
        sets.append([{i for i in range(bolt.bolt_num_instances(bolt.OP_CONV2D)) if bolt.bolt_instance_supports(
            bolt.OP_CONV2D, i, Cd(n, h, h, c, 256, r, r, stride, r // 2))} for n in (1, 2, 8, 32, 128)])
    for found in sets:
        assert found[0] and all(ids == found[0] for ids in found[1:]), found


def test_workspace_bytes(bolt):
    d = bolt.conv_desc(32, 7, 7, 512, 512, 3, 3, 1, 1)
    assert bolt.bolt_workspace_bytes(bolt.OP_CONV2D, d, None, {"kernel_id": 0, "split_k": 4}) == 4 * 1568 * 512 * 4
    assert bolt.bolt_workspace_bytes(bolt.OP_CONV2D, d, None, {"kernel_id": 0, "split_k": 1}) == 0
    assert bolt.bolt_workspace_bytes(bolt.OP_CONV2D, d) >= 4 * 1568 * 512 * 4
    big = bolt.conv_desc(32, 56, 56, 64, 64, 3, 3, 1, 1)
    assert bolt.bolt_workspace_bytes(bolt.OP_CONV2D, big) == 0  # enough tiles: split-K is never tried


def test_status_strings(bolt):
    seen = {bolt.bolt_status_string(i) for i in range(7)}
    assert len(seen) == 7 and "ok" in seen


def test_null_pointers_are_rejected_before_any_launch(bolt):
    lib = bolt.binding.raw()
    d = bolt.gemm_desc(64, 64, 64)
    assert lib.bolt_gemm_epilogue(ctypes.byref(d), None, None, None, None, None, None, 0, None) == INVALID
    c = bolt.conv_desc(1, 8, 8, 8, 8, 3, 3, 1, 1)
    assert lib.bolt_conv2d_fprop_nhwc(ctypes.byref(c), None, None, None, None, None, None, 0, None) == INVALID
    assert lib.bolt_gemm_epilogue(ctypes.byref(d), 16, 32, None, 8, None, None, 0, None) == ALIGNMENT  # D misaligned
    assert lib.bolt_pad_channels_nhwc(None, None, 4, 3, 8, None) == INVALID
    assert lib.bolt_pad_channels_nhwc(16, 32, 4, 3, 7, None) == ALIGNMENT
    assert lib.bolt_pad_channels_nhwc(16, 32, 4, 9, 8, None) == INVALID
    assert lib.bolt_gemm_epilogue_residual(ctypes.byref(d), 16, 32, None, None, 64, 1.0, 48, None, None, 0, None) == INVALID
    assert lib.bolt_gemm_epilogue_residual(ctypes.byref(d), 16, 32, None, 64, 32, 1.0, 48, None, None, 0, None) == INVALID  # ldc < N
    assert lib.bolt_gemm_epilogue_residual(ctypes.byref(d), 16, 32, None, 72, 64, 1.0, 48, None, None, 0, None) == ALIGNMENT
    assert lib.bolt_conv2d_fprop_nhwc_residual(ctypes.byref(c), 16, 32, None, None, 1.0, 48, None, None, 0, None) == INVALID
    g0, g1 = bolt.gemm_desc(64, 64, 64, b_layout=bolt.LAYOUT_NK), bolt.gemm_desc(64, 64, 64, b_layout=bolt.LAYOUT_NK)
    r = lambda C_, ldc, D_: lib.bolt_b2b_gemm_residual(ctypes.byref(g0), ctypes.byref(g1), 16, 32, None, 48, None, C_, ldc, 1.0,
                                                       D_, None, None, 0, None)
    assert r(None, 64, 80) == INVALID      # no residual matrix
    assert r(64, 32, 80) == INVALID        # ldc < N1
    assert r(64, 68, 80) == ALIGNMENT      # ldc not a multiple of 8
    assert r(72, 64, 80) == ALIGNMENT      # residual pointer not 16-byte aligned
    c0, c1 = bolt.conv_desc(1, 8, 8, 8, 64, 3, 3, 1, 1), bolt.conv_desc(1, 8, 8, 64, 64, 1, 1, 1, 0)
    assert lib.bolt_b2b_conv_residual(ctypes.byref(c0), ctypes.byref(c1), 16, 32, None, 48, None, None, 1.0, 80, None, None, 0,
                                      None) == INVALID
    c1bad = bolt.conv_desc(1, 8, 8, 64, 64, 3, 3, 1, 1)
    assert lib.bolt_b2b_conv_residual(ctypes.byref(c0), ctypes.byref(c1bad), 16, 32, None, 48, None, 64, 1.0, 80, None, None, 0,
                                      None) == ILLEGAL
    assert lib.bolt_nchw_to_nhwc(None, 32, 1, 3, 8, 8, 8, None) == INVALID
    assert lib.bolt_nchw_to_nhwc(16, 32, 1, 3, 8, 8, 7, None) == ALIGNMENT      # C_padded % 8
    assert lib.bolt_nchw_to_nhwc(16, 40, 1, 3, 8, 8, 8, None) == ALIGNMENT      # NHWC side misaligned
    assert lib.bolt_nchw_to_nhwc(16, 32, 1, 9, 8, 8, 8, None) == INVALID        # C_padded < C
    assert lib.bolt_nhwc_to_nchw(16, 32, 1, 3, 8, 8, 12, None) == ALIGNMENT
    assert lib.bolt_nhwc_to_nchw(16, 32, 70000, 3, 8, 8, 8, None) == UNSUPPORTED
    assert lib.bolt_bias_act(None, None, 4, 8, 8, 1.0, 1.0, 1, None) == INVALID
    assert lib.bolt_bias_act(32, None, 4, 12, 16, 1.0, 1.0, 1, None) == ALIGNMENT
    assert lib.bolt_bias_act(32, None, 4, 16, 8, 1.0, 1.0, 1, None) == INVALID    # ldd < N
    assert lib.bolt_bias_act(32, None, 4, 8, 8, 1.0, 1.0, 9, None) == INVALID     # unknown activation
    assert lib.bolt_tune(0, None, None, None, None, 0, None, None, None, None) == INVALID


def test_pingpong_kernels_keep_their_working_set_in_registers():
    # The ping-pong kernel budgets its 256 registers per lane by hand (128 accumulators, 96 fragment registers, one
    # register of loader state per row); a version that spills more than a handful of registers outside the k loop has
    # lost that budget and with it the overlap the kernel is built for.  (Correctness does not depend on it: spill
    # traffic only makes the kernel's s_waitcnt vmcnt(N) waits more conservative, because loads complete in order.)
    # The build writes the compiler's per-kernel resource report next to the objects; the check is skipped where only
    # the built library was shipped.
    import glob
    import os
    build = os.path.join(os.path.dirname(__file__), "..", "paper_2110_15238_amd", "csrc", "_build")
    reports = glob.glob(os.path.join(build, "*.usage"))
    if not reports:
        pytest.skip("no build directory (library shipped pre-built)")
    seen = 0
    for path in reports:
        name = None
        for line in open(path):
            line = line.strip()
            if line.startswith("Function Name:"):
                name = line.split(":", 1)[1].strip()
            elif line.startswith("ScratchSize") and name and "fprop_pp_kernel" in name:
                seen += 1
                assert int(line.rsplit(":", 1)[1]) <= 128, (name, line)
    assert seen >= 4  # GEMM and convolution instance, each with and without the residual epilogue


def test_streaming_chains_are_compiled_apart_from_the_tiled_ones():
    """The out-of-line activation is compiled once per file, for the register budget of all its callers there: beside the
    streaming kernels 40 of the 91 kernels of the tiled chains came out with other registers.  Skipped as above."""
    import glob
    import os
    reports = glob.glob(os.path.join(os.path.dirname(__file__), "..", "paper_2110_15238_amd", "csrc", "_build", "*.usage"))
    if not reports:
        pytest.skip("no build directory (library shipped pre-built)")
    held = [{k for k in ("chain_stream_kernel", "b2b_chain_kernel", "b2b_chain_halo_kernel") if k in open(path).read()} for path in reports]
    assert {"chain_stream_kernel"} in held and {"b2b_chain_kernel", "b2b_chain_halo_kernel"} in held
    assert sum(map(len, held)) == 3


def test_objects_depend_on_every_header_and_on_the_flags():
    """make's own plan (nothing is run): each header and the Makefile, whose flags differ by file, send every kernel file to the compiler."""
    import subprocess
    csrc = os.path.join(ROOT, "paper_2110_15238_amd", "csrc")
    sources = sorted(f for f in os.listdir(csrc) if f.endswith(".hip"))
    for changed in sorted(f for f in os.listdir(csrc) if f.endswith(".hpp")) + ["Makefile"]:
        plan = subprocess.run(["make", "-n", "-W", changed, "lib"], cwd=csrc, capture_output=True, text=True, check=True).stdout
        compiled = sorted(set(re.findall(r" -c (\S+\.hip) ", plan)))
        assert compiled == sources, (changed, set(sources) - set(compiled))


def test_every_file_with_the_shared_main_loop_keeps_matrix_results_in_vector_registers():
    """dma_main_loop has several ends; with accumulation registers the compiler copies the accumulators from one to the other, which short
    reductions don't make up for (NCHW outputs of 1x1 filters over 40 to 200 channels: 3 to 7 %).  Skipped as above."""
    import subprocess
    csrc = os.path.join(ROOT, "paper_2110_15238_amd", "csrc")
    if not os.path.exists(os.path.join(csrc, "_build")):
        pytest.skip("no build directory (library shipped pre-built)")
    plan = subprocess.run(["make", "-n", "-W", "Makefile", "lib"], cwd=csrc, capture_output=True, text=True, check=True).stdout
    lines = {m.group(1): m.group(0) for m in re.finditer(r"^hipcc .* -c (\S+)\.hip .*$", plan, re.M)}
    held = {f for f in lines if re.search("fprop_dma_kernel|b2b_dma_kernel|b2b_chain_kernel", open(os.path.join(csrc, "_build", f + ".usage")).read())}
    assert {"inst_conv", "inst_gemm_nk", "inst_b2b_gemm_dma"} <= held
    assert all("-amdgpu-mfma-vgpr-form=1" in lines[f] for f in held), [f for f in held if "vgpr-form" not in lines[f]]


def test_even_channel_kernels_keep_their_workgroups_per_compute_unit():
    """512 registers per SIMD lane: tiles of up to 12 fragments run on four waves per SIMD, as their estimate in the pick rule counts
    (128 registers), those of one channel fragment on six (80), of four pixel fragments on eight (64).  Skipped as above."""
    report = os.path.join(ROOT, "paper_2110_15238_amd", "csrc", "_build", "inst_conv_even.usage")
    if not os.path.exists(report):
        pytest.skip("no build directory (library shipped pre-built)")
    found = re.findall(r"conv_even_kernelILi(\d+)ELi(\d+)ELi(\d+)E\S*\s+VGPRs: (\d+)\s+ScratchSize \[bytes/lane\]: (\d+)", open(report).read())
    assert len(found) >= 32
    for _, fm, fn, regs, scratch in (map(int, f) for f in found):
        most = (64 if fm <= 4 else 80) if fn == 1 else 128 if fm * fn <= 12 else 256
        assert regs <= most and scratch == 0, (fm, fn, regs, scratch)


def test_wide_fused_pairs_request_their_bias_ahead(tmp_path):
    """The last epilogue of a pair with 129 to 256 output columns has 32 bias quads per lane.  Each loaded where it is used is a round trip of
    its own (2.5 us per workgroup): a load with a wait for everything behind it and no other load between.  Skipped as above."""
    import subprocess
    tools = "/opt/rocm/llvm/bin/"
    build = os.path.join(ROOT, "paper_2110_15238_amd", "csrc", "_build")
    objects = [os.path.join(build, o) for o in ("inst_b2b_gemm_dma.o", "inst_b2b_conv_dma.o")]
    if not all(map(os.path.exists, objects + [tools + "llvm-objdump"])):
        pytest.skip("no build directory or no disassembler")
    seen = 0
    for o in objects:
        fat, code = str(tmp_path / "fat"), str(tmp_path / "code")
        subprocess.check_call([tools + "llvm-objcopy", "--dump-section", ".hip_fatbin=" + fat, o, str(tmp_path / "copy")])
        subprocess.check_call([tools + "clang-offload-bundler", "--type=o", "--unbundle", "--input=" + fat, "--output=" + code,
                               "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"])
        listing = subprocess.run([tools + "llvm-objdump", "-d", "-C", "--no-show-raw-insn", code], capture_output=True, text=True, check=True).stdout
        for part in re.split(r"\n(?=[0-9a-f]+ <)", listing):
            kernel = re.match(r"[0-9a-f]+ <void bolt::b2b_dma_kernel<\d+, \d+, \d+, \d+, 256, ", part)
            if not kernel:
                continue
            events = re.findall(r"^\s+(global_load_\w+|buffer_load_\w+|s_waitcnt [^\n/]*vmcnt\(\d+\))", part, re.M)
            alone = sum(1 for before, load, wait in zip(events, events[1:], events[2:])
                        if "vmcnt(0)" in wait and load.startswith("global_load") and "vmcnt(0)" in before)
            seen += 1
            assert alone <= 8, (kernel.group(0), alone)
    assert seen >= 8


def test_pick_rule_counts_the_activations_of_tall_thin_problems():
    """The kernels for small problems may not be estimated below the time that reading the activations takes: thousands of
    rows times a deep reduction, where the tiled kernels are up to 1.4 times faster.  Small problems stay with them."""
    import os
    import re
    import subprocess
    import sys
    code = """
import sys
sys.path.insert(0, %r)
import paper_2110_15238_amd as b
for m, n, k in ((16384, 8, 8192), (16384, 16, 8192), (16384, 32, 8192), (8192, 64, 2048), (32, 1000, 2048)):
    for layout in (b.LAYOUT_KN, b.LAYOUT_NK):
        assert b.bolt_check(b.OP_GEMM, b.gemm_desc(m, n, k, b_layout=layout)) == 0
""" % os.path.abspath(ROOT)
    r = subprocess.run([sys.executable, "-c", code], env=dict(os.environ, BOLT_TUNE_LOG="1"), capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    picks = re.findall(r"\[bolt_pick\] -> \d+ (\S+)", r.stderr)
    assert len(picks) == 10 and not any(p.startswith("ws_") for p in picks[:8]) and all(p.startswith("ws_") for p in picks[8:]), picks
    costs = [float(c) for c in re.findall(r"candidate \d+ ws_\S+ cost (\S+)", r.stderr.split("->")[0])]
    assert costs and min(costs) >= 2 * 16384 * 8192 / 6.5e6, costs  # the activations at 6.5 TB/s


def test_calls_without_the_extension_take_the_general_path():
    """An interpreter or torch that cannot load _fastcall: the package imports, the first call says so once, and every launch call
    is marshalled (here: refused, the tensors are on the CPU) through ctypes."""
    import os
    import subprocess
    import sys
    code = """
import sys, warnings
sys.path.insert(0, %r)
sys.modules["paper_2110_15238_amd._fastcall"] = None  # as if it could not be loaded
import torch
import paper_2110_15238_amd as b
t = torch.zeros(64, 64, dtype=torch.float16)
d, c = b.gemm_desc(64, 64, 64), b.conv_desc(1, 8, 8, 64, 64, 1, 1)
calls = [lambda: b.bolt_gemm_epilogue(d, t, t, None, t), lambda: b.bolt_gemm_epilogue_residual(d, t, t, None, t, t),
         lambda: b.bolt_conv2d_fprop_nhwc(c, t, t, None, t), lambda: b.bolt_conv2d_fprop_nhwc_residual(c, t, t, None, t, t),
         lambda: b.bolt_b2b_gemm(d, d, t, t, None, t, None, t), lambda: b.bolt_b2b_conv(c, c, t, t, None, t, None, t),
         lambda: b.bolt_b2b_gemm_chain([d] * 3, t, [t] * 3, [None] * 3, t), lambda: b.bolt_b2b_conv_chain([c] * 3, t, [t] * 3, [None] * 3, t)]
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    refused = 0
    for call in calls:
        try:
            call()
        except AssertionError as e:
            refused += "CUDA float16" in str(e)
assert refused == len(calls), refused
assert [w.category for w in seen] == [RuntimeWarning], seen
""" % os.path.abspath(ROOT)
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]


def test_the_c_library_builds_without_torch():
    """`make lib`, and `make` where the Python has no torch, ask for nothing but hipcc (dry run: nothing is compiled)."""
    import os
    import subprocess
    csrc = os.path.join(os.path.abspath(ROOT), "paper_2110_15238_amd", "csrc")
    run = lambda *a: subprocess.run(["make", "-C", csrc, "-n", "-B", *a], capture_output=True, text=True, check=True).stdout
    assert "fastcall" not in run("lib") and "libbolt.so" in run("lib")
    assert "fastcall.cpp" not in run("PYTHON=false") and "libbolt.so" in run("PYTHON=false")
    assert "fastcall.cpp" in run()


def _picks(calls):
    """The kernels that the built-in rule picks for a list of expressions over `b`, the package (BOLT_TUNE_LOG=1 names them)."""
    import os
    import re
    import subprocess
    import sys
    code = "import sys\nsys.path.insert(0, %r)\nimport paper_2110_15238_amd as b\n" % os.path.abspath(ROOT)
    code += "\n".join("assert %s == 0" % c for c in calls)
    r = subprocess.run([sys.executable, "-c", code], env=dict(os.environ, BOLT_TUNE_LOG="1"), capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    picks = re.findall(r"\[bolt_pick\] -> \d+ (\S+)", r.stderr)
    assert len(picks) == len(calls), picks
    return picks


def test_pairs_stream_where_their_rounds_are_full_or_activations_cheap():
    """Streaming pairs cost up to 1.9 times the tiled ones with GELU or a short last round; (64, 32) and full rounds gain."""
    def pair(m, k0, n0, n1, a0, a1):
        return "b.bolt_check(b.OP_B2B_GEMM, b.gemm_desc(%d, %d, %d, act=%r), b.gemm_desc(%d, %d, %d, act=%r))" % (m, n0, k0, a0, m, n1, n0, a1)
    tiled = [pair(78392, 32, 24, 48, "gelu", "gelu"), pair(78392, 32, 24, 48, "relu", "relu"), pair(66211, 96, 16, 72, "relu", "relu"),
             pair(152820, 48, 8, 104, "relu", "relu"), pair(109942, 48, 8, 104, "gelu", "gelu"), pair(68365, 80, 16, 16, "gelu", "none"),
             pair(78816, 40, 64, 64, "gelu", "gelu"), pair(65536, 96, 64, 32, "relu", "relu")]
    streamed = [pair(131072, 96, 64, 32, "relu", "relu"), pair(74538, 96, 64, 32, "gelu", "gelu"), pair(78816, 40, 64, 64, "relu", "hardswish"),
                pair(109000, 40, 64, 64, "gelu", "gelu"), pair(109942, 48, 8, 104, "relu", "relu"), pair(120995, 40, 128, 64, "softplus", "softplus"),
                pair(67914, 24, 56, 120, "gelu", "gelu")]
    picks = _picks(tiled + streamed)
    assert [p.startswith("pairstream") for p in picks] == [False] * len(tiled) + [True] * len(streamed), picks
    assert picks[len(tiled)].endswith("n64_32") and picks[len(tiled) + 3].endswith("n64_64")


def test_chains_with_heavy_activations_stream_only_in_full_rounds():
    """Where two tiled workgroups fit on a compute unit; with one (64, 128, 64) the streaming kernel always gains."""
    def chain(m, widths, *acts):
        return "b.bolt_check_chain(b.OP_GEMM_CHAIN3, [%s])" % ", ".join(
            "b.gemm_desc(%d, %d, %d, act=%r)" % (m, n, k, a) for k, n, a in zip(widths, widths[1:], acts))
    tiled = [chain(69774, (48, 48, 48, 48), "gelu", "gelu", "gelu"), chain(69774, (48, 48, 48, 48), "none", "none", "softplus"),
             chain(83006, (8, 48, 16, 8), "relu", "relu", "relu"), chain(65536, (48, 48, 48, 48), "hardswish", "relu", "relu")]
    streamed = [chain(69774, (48, 48, 48, 48), "relu", "hardswish", "none"), chain(110000, (48, 48, 48, 48), "gelu", "gelu", "gelu"),
                chain(69100, (40, 64, 72, 56), "gelu", "gelu", "gelu"), chain(128320, (96, 32, 96, 32), "relu", "relu", "relu")]
    picks = _picks(tiled + streamed)
    assert [p.startswith("chainstream") for p in picks] == [False] * len(tiled) + [True] * len(streamed), picks


def test_deep_reductions_over_many_small_tiles_stay_with_the_tiled_kernels():
    """More than 256 tiles of 32 x 32: the kernels for small problems are up to 1.45 times slower with a deep reduction, faster with a short one."""
    gemm = lambda m, n, k, lay: "b.bolt_check(b.OP_GEMM, b.gemm_desc(%d, %d, %d, b_layout=b.LAYOUT_%s))" % (m, n, k, lay)
    conv = lambda *a: "b.bolt_check(b.OP_CONV2D, b.conv_desc%r)" % (a,)
    tiled = [gemm(4677, 40, 3272, "KN"), gemm(2986, 80, 2000, "NK"), gemm(759, 608, 4784, "KN"), conv(1, 56, 56, 1568, 128, 1, 1),
             conv(3, 14, 14, 408, 648, 3, 3, 1, 1)]
    split = [gemm(989, 440, 384, "KN"), gemm(32, 1000, 2048, "KN"), conv(12, 7, 7, 40, 504, 5, 5, 1, 2), conv(7, 28, 28, 40, 48, 5, 5, 1, 2)]
    picks = _picks(tiled + split)
    assert [p.startswith("ws_") for p in picks] == [False] * len(tiled) + [True] * len(split), picks


def test_one_tap_filters_over_many_unpadded_pixels_stay_with_the_alignment_2_kernels():
    """1x1 filters give nothing to the patch in LDS that kernels for unpadded channels copy: above 16000 input pixels and 32 channels."""
    conv = lambda *a: "b.bolt_check(b.OP_CONV2D, b.conv_desc%r)" % (a,)
    picks = _picks([conv(80, 30, 28, 98, 40, 1, 1, 2), conv(88, 36, 18, 34, 64, 1, 1, 2), conv(2, 59, 27, 82, 16, 1, 1, 2), conv(46, 28, 10, 114, 32, 1, 1),
                    conv(128, 14, 19, 46, 32, 5, 7)])
    assert [p.startswith("even_") for p in picks] == [False, False, True, True, True], picks


def test_pairs_keep_to_the_tiled_kernels_where_images_do_not_fill_units():
    """conv_patch_kernel works on 4 x 8 output pixels of one image: many images of one column or one pixel took it up to 14 times as
    long as the tiled kernels.  Elsewhere it gains, also with units that are half full where the tiled kernels' widths do not fit."""
    def pair(n, h, w, c, k0, r, stride, k1):
        p, q = (h - 1) // stride + 1, (w - 1) // stride + 1
        return ("b.bolt_check(b.OP_B2B_CONV, b.conv_desc(%d, %d, %d, %d, %d, %d, %d, %d, %d), b.conv_desc(%d, %d, %d, %d, %d, 1, 1))" %
                (n, h, w, c, k0, r, r, stride, r // 2, n, p, q, k0, k1))
    tiled = [pair(100000, 1, 1, 64, 64, 3, 1, 256), pair(12000, 1, 1, 64, 64, 1, 1, 256), pair(1785, 56, 1, 32, 32, 3, 1, 64), pair(166, 300, 2, 64, 64, 3, 2, 128),
             pair(25000, 2, 2, 128, 64, 1, 1, 64), pair(1785, 1, 56, 64, 64, 3, 1, 256)]
    patch = [pair(1000, 1, 1, 64, 64, 3, 1, 256), pair(32, 56, 56, 64, 64, 3, 1, 256), pair(214, 7, 56, 32, 32, 3, 1, 128), pair(32, 112, 112, 32, 32, 3, 1, 64),
             pair(2040, 7, 7, 64, 64, 1, 1, 256), pair(4, 14, 14, 64, 64, 3, 1, 256), pair(32, 56, 56, 64, 64, 3, 2, 32),
             pair(72, 85, 11, 56, 16, 3, 1, 72), pair(179, 19, 86, 64, 56, 1, 2, 8)]  # (half-filled units, but tiled kernels of twice to four times the width)
    picks = _picks(tiled + patch)
    assert [p.startswith("b2bpatch_") for p in picks] == [False] * len(tiled) + [True] * len(patch), picks


def test_small_3x3s_stay_with_the_kernels_for_small_problems():
    """The streamed and the sliced 3x3 kernels, one round of units or tiles: not where the wave-split kernels are faster."""
    conv = lambda n, h, w, c, k: "b.bolt_check(b.OP_CONV2D, b.conv_desc(%d, %d, %d, %d, %d, 3, 3, 1, 1))" % (n, h, w, c, k)
    small = [conv(550, 1, 1, 8, 32), conv(4, 3, 3, 16, 16), conv(30, 22, 4, 24, 16), conv(172, 1, 26, 40, 32), conv(27, 48, 1, 64, 64), conv(20, 8, 3, 128, 152)]
    new = [conv(22, 25, 8, 32, 64), conv(7, 57, 36, 8, 16), conv(119, 25, 12, 8, 48), conv(8, 56, 56, 64, 64), conv(8, 28, 28, 128, 128), conv(6, 10, 25, 128, 64)]
    picks = _picks(small + new)
    assert [p.split("_")[0] for p in picks] == ["ws"] * len(small) + ["patch"] * 4 + ["slice"] * 2, picks


def test_built_in_pick_rule_families():
    """What a call without a config runs (no GPU needed: bolt_check resolves the pick, BOLT_TUNE_LOG=1 names it): the
    halo kernel for a 3x3 stride-1 layer, the ping-pong kernels for a GEMM that fills the chip in either weight layout,
    the direct-to-LDS kernel (never its register-staged cover) for row-major weights, 32-deep k-tiles for K = 32."""
    import os
    import re
    import subprocess
    import sys
    root = os.path.join(os.path.dirname(__file__), "..")
    code = """
import sys
sys.path.insert(0, %r)
import paper_2110_15238_amd as b
cases = [(b.OP_CONV2D, b.conv_desc(32, 56, 56, 64, 64, 3, 3, 1, 1)),
         (b.OP_GEMM, b.gemm_desc(4096, 4096, 4096, b_layout=b.LAYOUT_NK)),
         (b.OP_GEMM, b.gemm_desc(4096, 4096, 4096)),
         (b.OP_GEMM, b.gemm_desc(1280, 768, 3072)),
         (b.OP_GEMM, b.gemm_desc(128320, 96, 32))]
for op, d in cases:
    assert b.bolt_check(op, d) == 0
""" % os.path.abspath(root)
    r = subprocess.run([sys.executable, "-c", code], env=dict(os.environ, BOLT_TUNE_LOG="1"), capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    picks = re.findall(r"\[bolt_pick\] -> \d+ (\S+)", r.stderr)
    assert len(picks) == 5, picks
    assert picks[0].startswith("halo_")
    assert picks[1].startswith("pp_") and picks[2].startswith("ppkn_")
    assert picks[3].startswith("dmakn_")
    assert picks[4].startswith("dmakn_") and re.match(r"dmakn_\d+x\d+x32_", picks[4])

