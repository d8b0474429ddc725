"""Which kernel, division and workspace a call gets (the host's choice; no GPU): the library's
host code compiled on its own, asked for 256 compute units."""
import ctypes
import os
import subprocess

import pytest

import workloads as W

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")
pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
FIELDS = "total rgen tall narrow fused S F p16 vsplit sk_slots nplans".split()
MIB, GIB = 1 << 20, 1 << 30


@pytest.fixture(scope="module")
def layout(tmp_path_factory):
    import paper_2609_32922_amd._lib as L
    out = str(tmp_path_factory.mktemp("layout") / "layout.so")
    # (only the query is exported, so the entry points and the launches they call fall away)
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
                        "-Xarch_host", "-ffunction-sections", "-Wl,--gc-sections", "-Xclang", "-target-feature",
                        "-Xclang", "-packed-fp32-ops", os.path.join(HERE, "layout_query.hip"), "-o", out],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    lib = ctypes.CDLL(out)
    lib.layout_query.argtypes = [ctypes.POINTER(L.ScGemmDesc), ctypes.c_int, ctypes.c_int, ctypes.POINTER(ctypes.c_int64)]

    def ask(batch, M, N, K, L_max, polarity=0, hint=0, rng=0, own_B=False, tables=False, **kw):
        d = L.ScGemmDesc()
        d.batch, d.M, d.N, d.K, d.lda, d.ldb, d.ldo = batch, M, N, K, K, K, N
        d.strideA, d.strideB, d.strideO = M * K, N * K if own_B else 0, M * N
        d.strideSA, d.strideSB, d.strideL = M, N if own_B else 0, M
        d.L_max, d.polarity, d.rng, d.L_hint = L_max, polarity, rng, hint
        for k, v in kw.items():
            setattr(d, k, v)
        o = (ctypes.c_int64 * len(FIELDS))()
        rc = lib.layout_query(ctypes.byref(d), 256, int(tables), o)
        return dict(zip(FIELDS, o)) if rc == 0 else rc

    return ask


@pytest.mark.parametrize("batch,M,K,L_max,polarity,parts", [
    (16, 8224, 64, 256, 0, 1),       # the compensator: 32 rows, ten steps
    (256, 550, 577, 256, 1, 1),
    (16, 8320, 256, 256, 0, 8),      # 128 rows, 40 steps a tile
    (128, 1152, 577, 256, 0, 4),
    (64, 2115, 256, 512, 1, 8),
])
def test_ragged_last_round_of_narrow_tiles(layout, batch, M, K, L_max, polarity, parts):
    # 256 x 64 blocks, one length: a last round of half-filled tiles stays whole only while it is short
    lay = layout(batch, M, 64, K, L_max, polarity)
    assert lay["narrow"] and lay["S"] == parts


@pytest.mark.parametrize("batch,M,N,K,L_max,hint,own_B,most", [
    (1, 406072, 87105, 5304, 1579, 700, False, 137 * GIB),      # (217 with the lighter steps' ranges)
    (1, 1060669, 42937, 342, 2277, 1000, False, 18 * GIB),      # (27)
    (16, 17882, 29643, 22308, 2554, 851, False, 224 * GIB),     # tiles longer than one range may hold (353)
    (1, 1098945, 12731, 8310, 3703, 370, True, 202 * GIB),
])
def test_workspace_of_long_range_divisions(layout, batch, M, N, K, L_max, hint, own_B, most):
    lay = layout(batch, M, N, K, L_max, hint=hint, own_B=own_B)
    assert lay["vsplit"] and lay["total"] <= most
    # every range's steps stay exact where a tile alone has more
    KC, G = (K + 31) // 32, (L_max + 31) // 32
    tiles = batch * ((M + 255) // 256) * ((N + 255) // 256)
    if KC * G > 1 << 14:
        assert -(-tiles * (KC * G + 7) // lay["sk_slots"]) + 2 <= 1 << 14


@pytest.mark.parametrize("batch,M,N,K,L_max,hint,own_B,accepted", [
    (128, 5815, 50232, 27389, 1039, 103, False, True),
    (1, 2966264, 7154, 26588, 1463, 146, False, True),
    (13, 101552, 12575, 86011, 768, 76, True, True),
    (1, 1 << 21, 1 << 21, 1 << 15, 4096, 100, False, False),
])
def test_range_division_limit(layout, batch, M, N, K, L_max, hint, own_B, accepted):
    # 2^20 ranges of 2^14 steps, whatever a step weighs (no card holds these calls: only the answer matters)
    lay = layout(batch, M, N, K, L_max, hint=hint, own_B=own_B)
    assert isinstance(lay, dict) == accepted and (accepted or lay == -2)


@pytest.mark.parametrize("batch,M,N,K,own_B,most", [
    (815, 1, 29, 7782, False, 520 * MIB),        # (1.6 GiB with A's chunks in whole pairs of 256 rows)
    (815, 1, 29, 7782, True, 910 * MIB),         # (B's too: 3.1)
    (128, 100, 100, 768, True, 33 * MIB),         # (56)
    (1, 48, 3072, 768, False, 10 * MIB),
])
def test_workspace_of_few_rows_and_columns(layout, batch, M, N, K, own_B, most):
    # chunks of the 64 (128) rows and columns that 64-row blocks read, and not of 256
    lay = layout(batch, M, N, K, 64, own_B=own_B)
    assert lay["tall"] and lay["total"] <= most


@pytest.mark.parametrize("batch,M,N,K,L_max,polarity,own_B,grows", [
    (1, 6304, 3072, 768, 128, 0, False, 1 * MIB),       # (34 MiB beside planes of 499)
    (1, 381, 287391, 21327, 81, 1, False, 1 * MIB),     # (8 GiB beside planes of 275)
    (1, 1645729, 679, 3987, 82, 0, False, 1 * MIB),     # (6 GiB beside 270)
    (16, 325, 1091, 2000, 96, 1, True, 1 * MIB),
    (24, 8224, 64, 130, 256, 0, True, 1 * MIB),
    (1000, 129, 64, 500, 128, 0, True, 1 * MIB),
])
def test_workspace_of_cbsg_tables(layout, batch, M, N, K, L_max, polarity, own_B, grows):
    # the tables lie where the planes will if they do not serve
    planes = layout(batch, M, N, K, L_max, polarity, rng=1, own_B=own_B)
    tables = layout(batch, M, N, K, L_max, polarity, rng=1, own_B=own_B, tables=True)
    assert planes["total"] <= tables["total"] <= planes["total"] + grows


def test_cbsg_tables_over_every_planes_layout(layout):
    # each part of the tables inside the planes' part it lies on: over sizes where either is tightest
    n = 0
    for K in (1, 3, 16, 17, 33, 64, 97, 1000):
        for L_max in (9, 16, 17, 33, 64, 255, 256):
            for M, N in ((1, 1 << 20), (64, 70000), (100, 40000), (129, 60), (300, 300), (70000, 100), (1 << 20, 1)):
                batch = max(1, int(4.1e11 // (M * N * K * L_max)) + 1)
                if batch > 1 << 20:
                    continue
                lay = layout(batch, M, N, K, L_max, rng=1, own_B=True, tables=True)
                if isinstance(lay, dict):
                    n += 1
                    planes = layout(batch, M, N, K, L_max, rng=1, own_B=True)
                    assert lay["total"] <= planes["total"] * 1.01 + MIB, (batch, M, N, K, L_max)
    assert n > 100


@pytest.mark.parametrize("batch,M,N,K,L_max,hint,fused", [
    (564, 79, 128, 378, 7, 0, True),         # few rows each: both operands' chunks, 67 us against 93
    (49666, 16, 4, 268, 4, 1, True),
    (51261, 8, 68, 266, 8, 2, True),         # 2.9 ms against 4.2
    (209, 16, 128, 1441, 1, 0, False),       # 82 us against 67
    (830, 339, 100, 124, 9, 3, True),        # lengths of 9 and less: 109 us against 137
    (616, 108, 32, 4609, 24, 8, False),      # 912 us against 640
    (1, 24589, 116, 1983, 8, 0, True),
    (8, 45067, 87, 3067, 8, 0, True),
    (1, 40413, 118, 2959, 16, 5, True),
    (1, 2196, 114, 71, 8, 2, False),
    (8, 3811, 79, 1032, 16, 8, False),
    (1, 24589, 116, 400, 64, 0, False),
])
def test_few_columns_and_short_streams(layout, batch, M, N, K, L_max, hint, fused):
    # an octet of cycles costs 64-row blocks a whole group of 32 slots: k_fgemm where the call is large
    lay = layout(batch, M, N, K, L_max, hint=hint, own_B=batch > 100)
    assert bool(lay["fused"]) == fused and bool(lay["tall"]) != fused


ARRAY = 64 * MIB      # sc_gemm_noalloc's


@pytest.mark.parametrize("batch,M,N,K,L_max,hint,own_B,fused", [
    (18, 637, 100, 4669, 12, 4, True, True),      # 103 us against 175 in the parts that fit
    (2, 8521, 100, 3018, 16, 5, True, True),      # 115 against 135
    (61, 103, 63, 4915, 24, 8, True, False),      # 140 against 116
    (163, 97, 32, 1627, 12, 4, True, False),      # 117 against 81
])
def test_few_columns_past_the_array(layout, batch, M, N, K, L_max, hint, own_B, fused):
    lay = layout(batch, M, N, K, L_max, hint=hint, own_B=own_B)
    assert bool(lay["fused"]) == fused and lay["total"] <= ARRAY


@pytest.mark.parametrize("batch,M,N,K,L_max,polarity", [
    (1, 2200, 1024, 1024, 256, 0),       # 66.6 MiB in 7 parts
    (1, 577, 4096, 1024, 256, 0),
    (1, 514, 4608, 1152, 192, 1),
    (1, 1700, 1152, 4608, 192, 0),
    (1, 2669, 3969, 748, 128, 0),        # 131.6
    (1, 4815, 768, 768, 512, 0),         # 65 with the tables of all plans
    (512, 256, 72, 256, 192, 0),
])
def test_calls_near_the_array_keep_their_plans(layout, batch, M, N, K, L_max, polarity):
    lay = layout(batch, M, N, K, L_max, polarity)
    assert lay["total"] <= ARRAY and lay["nplans"] > 1 and lay["rgen"]


@pytest.mark.parametrize("N,K", [(768, 768), (3072, 768), (768, 3072), (1024, 1024), (4096, 1024), (1024, 4096),
                                 (1152, 1152), (4608, 1152), (1152, 4608)])
def test_no_row_count_loses_the_plans(layout, N, K):
    # one row length: the array never costs a call its plans (it did for 7 % of these)
    for L_max in (64, 128, 192, 256):
        for M in range(150, 8192, 97):
            lay = layout(1, M, N, K, L_max)
            assert lay["nplans"] > 1, (M, L_max, lay)


@pytest.mark.parametrize("L_max,tables", [(1, False), (4, False), (8, False), (9, True), (128, True)])
def test_cbsg_tables_from_an_octet_of_cycles_on(layout, L_max, tables):
    # a group of 32 slots for less than that costs more than the planes
    assert isinstance(layout(4, 13132, 5516, 768, L_max, 1, rng=1, tables=True), dict) == tables


def _cases(name):
    import test_gpu_parity
    return getattr(test_gpu_parity, name)


# (columns of a wave / 32, parts, int16 counts) that each case of 64-row blocks takes, in order
TALL_VARIANTS = [(1, 4, 1), (1, 1, 0), (1, 8, 1), (1, 8, 0), (5, 1, 0), (4, 7, 1), (1, 1, 0), (4, 5, 1), (5, 1, 0),
                 (2, 1, 0), (2, 8, 1), (2, 8, 1), (1, 1, 0), (1, 9, 0)]


def test_the_parity_cases_take_the_variants_they_name(layout):
    """A case whose sizes come to take another kernel or division is to be replaced, not kept under its label."""
    got = []
    for batch, M, N, K, L_max, _, pol, bcast, _ in _cases("TALL"):
        lay = layout(batch, M, N, K, L_max, pol, own_B=not bcast and batch > 1)
        got.append((lay["tall"], lay["S"], lay["p16"]))
    assert got == TALL_VARIANTS
    got = []
    for M, N, K, L_max, _, pol, _ in _cases("INT32_PARTS"):
        lay = layout(1, M, N, K, L_max, pol)
        got.append((lay["tall"], lay["S"], lay["p16"]))
    assert got == [(2, 8, 0), (2, 8, 0), (4, 8, 0), (4, 8, 0)]
    got = []
    for batch, M, N, K, L_max, _, pol, bcast, _ in _cases("FGEMM"):
        lay = layout(batch, M, N, K, L_max, pol, own_B=not bcast and batch > 1)
        got.append((lay["fused"], lay["S"]))
    assert got == [(1, 1), (1, 1), (1, 2), (1, 8), (1, 8), (1, 1)]
    assert layout(1, 40000, 70, 1500, 8, lda=1507, ldb=1503, ldo=75)["fused"]
    got = []
    for M, N, K, L_max, rng in _cases("PAST_BOUND"):
        lay = layout(1, M, N, K, L_max, rng=rng)
        got.append((lay["rgen"], lay["tall"], lay["narrow"], lay["S"] >= 2))
    assert got == [(1, 1, 0, True), (1, 1, 0, True), (1, 1, 0, True), (1, 0, 1, True), (1, 0, 0, True),
                   (0, 0, 0, True), (0, 0, 0, True)]
    for batch, M, N, K, L_max, kind, hint, pol, bcast, _ in _cases("WIDE"):
        lay = layout(batch, M, N, K, L_max, pol, hint=hint, own_B=not bcast and batch > 1)
        assert lay["rgen"] and not lay["tall"] and not lay["narrow"] and bool(lay["vsplit"]) == (hint > 0)
    for M, N, K, L_max, pol, _ in _cases("LONG_RANGES"):
        lay = layout(1, M, N, K, L_max, pol, hint=int(L_max * 0.66))
        assert lay["vsplit"] and not lay["narrow"]


def test_outputs_past_31_bit_offsets_take_parts(layout):
    for M, N, K, L_max in ((5, 70, 40, 64), (3, 300, 100, 96)):
        assert layout(1, M, N, K, L_max, ldo=(1 << 29) // (M - 2) + 9)["S"] >= 2


@pytest.mark.parametrize("name", sorted(W.WORKLOADS))
def test_benchmark_names_the_kernel_that_runs(layout, name):
    # the roofline's kernel name is worked out from the shape; the layout is what the call takes
    import bench
    for g in W.WORKLOADS[name]().gemms:
        hint = int(round(float(g.L.mean())))
        shape = dict(batch=g.batch, M=g.M, N=g.N, K=g.K, L_max=g.L_max, polarity=g.polarity, hint=hint,
                     own_B=g.B.shape[0] > 1)
        for rng in (0, 1):
            if rng == 1 and g.L_max > 256:
                continue
            lay = layout(rng=rng, **shape)
            if rng == 1 and g.L.min() == g.L_max:
                tables = layout(rng=1, tables=True, **shape)
                lay = tables if isinstance(tables, dict) else lay
            want = ("k_tgemm" if lay["tall"] else "k_rgemm_n" if lay["narrow"] else "k_rgemm") if lay["rgen"] else \
                   ("k_qgemm" if g.M > 128 and g.N > 128 else "k_mgemm")
            assert bench.gemm_kernel_name(g, rng == 0) == want, (name, g.name, rng)
