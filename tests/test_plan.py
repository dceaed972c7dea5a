"""Expert-GEMM plans (host logic, no GPU): the kernel family each workload shape
takes, and launch grids that cover every split of the rows into expert groups
(a grid short of the device-side tile count would leave tiles uncomputed)."""

import ctypes

import numpy as np
import pytest
import torch

from paper_2608_24938_amd import exfold as X

FAKE = 0x10000  # weights are never dereferenced by the planner
SIMT, TILE, SKINNY, WIDE = range(4)  # SIMT: the float32 layers


def layer(d, inter, n, k, shared=0, dtype=X.BF16):
    return X._Layer(d, inter, n, k, shared, dtype, 0, FAKE, None, FAKE, FAKE,
                    FAKE if shared else None, FAKE if shared else None)


def plan(ly, rows, active, cu=256):
    out = (ctypes.c_int32 * 10)()
    assert X.lib().exfold_gemm_plan(ctypes.byref(ly), rows, active, cu, out) == X.OK
    v = list(out)
    return dict(zip(("kind", "bm", "bn", "ksplit", "grid"), v[:5])), dict(zip(("kind", "bm", "bn", "ksplit", "grid"), v[5:]))


MIXTRAL = dict(d=4096, inter=14336, n=8, k=2)
QWEN3 = dict(d=2048, inter=768, n=128, k=8)
GLM = dict(d=4096, inter=1408, n=128, k=8, shared=1408)


@pytest.mark.parametrize("shape,rows,active,gu_kind,dn_kind", [
    (MIXTRAL, 4096, 8, WIDE, WIDE),          # prefill, 4096 tokens, K' = 1
    (MIXTRAL, 8192, 8, WIDE, WIDE),
    (MIXTRAL, 64, 4, SKINNY, SKINNY),        # decode, 32 tokens, pool of 4
    (QWEN3, 32768, 128, WIDE, WIDE),         # prefill, 8192 tokens, K' = 4
    (QWEN3, 1024, 16, TILE, TILE),           # decode, 128 tokens, pool of 16 (64 rows per expert)
    (QWEN3, 1024, 64, SKINNY, SKINNY),       # decode, 128 tokens, pool of 64 (16 rows per expert)
    (QWEN3, 4096, 32, WIDE, WIDE),           # decode, 512 tokens, pool of 32 (wide down without a full round)
    (QWEN3, 2048, 16, TILE, TILE),           # 128 rows per expert but 48 wide tiles, under a quarter round
    (QWEN3, 2048, 32, TILE, TILE),           # 64 rows per expert: 128x128 down tiles above 48 rows
    (QWEN3, 1024, 32, TILE, SKINNY),         # 32 rows per expert: skinny down tiles up to 48 rows
    (QWEN3, 512, 16, TILE, SKINNY),          # 32 rows per expert: 128x128 gate/up tiles above 24 rows
    (QWEN3, 384, 16, SKINNY, SKINNY),        # 24 rows per expert: skinny gate/up tiles
    (GLM, 64 * 8 + 64, 33, SKINNY, SKINNY),  # decode with the shared expert
    (GLM, 4096 * 4 + 4096, 129, TILE, TILE),  # I = 1408 splits into no 256-wide pairs
])
def test_kernel_family(shape, rows, active, gu_kind, dn_kind):
    gu, dn = plan(layer(**shape), rows, active)
    assert (gu["kind"], dn["kind"]) == (gu_kind, dn_kind), (gu, dn)


# One range: the rows travel as bf16.  More: as float32 partials.  An intermediate size that is an odd multiple
# of 64 is split as its count of 128 x 128 tiles asks for, on whatever tiles it runs.
@pytest.mark.parametrize("d,inter,n,active,rows,ksplit", [
    (512, 1728, 64, 34, 1598, 3), (7168, 4160, 8, 2, 16, 5), (7168, 14400, 8, 4, 16, 3), (640, 6720, 65, 13, 319, 7),
    (512, 4800, 49, 28, 80, 5), (4480, 4928, 2, 1, 1, 7), (640, 960, 8, 1, 4, 1),
    (7168, 4096, 8, 2, 16, 4), (4096, 14336, 8, 4, 64, 2),   # even multiples: three 32 x 64 tiles a CU
])
def test_down_split(d, inter, n, active, rows, ksplit):
    _, dn = plan(layer(d, inter, n, 1), rows, active)
    assert dn["ksplit"] == ksplit, dn
    assert inter // 64 % ksplit == 0


# Skinny tiles: 32 rows up to 12 rows a busy expert, and up to 24 where there are at most four tiles a CU; else 64.
@pytest.mark.parametrize("shape,rows,active,gu_bm,dn_bm", [
    (QWEN3, 12 * 64, 64, 32, 32), (QWEN3, 12 * 64 + 1, 64, 64, 64), (QWEN3, 12 * 128 + 1, 128, 64, 64),
    (MIXTRAL, 96, 8, 32, 32), (MIXTRAL, 97, 8, 64, 32), (MIXTRAL, 24 * 8, 8, 64, 32), (MIXTRAL, 24 * 8 + 1, 8, 128, 64),
    (dict(d=1024, inter=512, n=32, k=4), 720, 32, 32, 32), (dict(d=1024, inter=512, n=32, k=4), 769, 32, 128, 64),
    (dict(d=2048, inter=768, n=32, k=4), 640, 32, 32, 32), (dict(d=2048, inter=1088, n=32, k=4), 640, 32, 64, 32),
])
def test_skinny_tile_height(shape, rows, active, gu_bm, dn_bm):
    gu, dn = plan(layer(**shape), rows, active)
    assert (gu["bm"], dn["bm"]) == (gu_bm, dn_bm), (gu, dn)


# Down tiles: skinny up to 48 rows a busy expert, or 20 where there are more than two 128-column tiles a CU, and
# never for a reduction below one skinny stage (I = 64); else 128 columns, 64 rows a tile up to 80.  Gate/up:
# skinny up to 24 rows.
@pytest.mark.parametrize("d,inter,active,rows,gu,dn", [
    (2048, 768, 32, 24 * 32, (SKINNY, 32), (SKINNY, 32)), (2048, 768, 32, 24 * 32 + 1, (TILE, 128), (SKINNY, 64)),
    (2048, 768, 32, 48 * 32, (TILE, 128), (SKINNY, 64)), (2048, 768, 32, 48 * 32 + 1, (TILE, 128), (TILE, 64)),
    (2048, 768, 32, 80 * 32, (TILE, 128), (TILE, 64)), (2048, 768, 32, 80 * 32 + 1, (TILE, 128), (TILE, 128)),
    (2048, 768, 33, 20 * 33, (SKINNY, 32), (SKINNY, 64)), (2048, 768, 33, 20 * 33 + 1, (SKINNY, 32), (TILE, 64)),
    (256, 64, 4, 4, (SKINNY, 32), (TILE, 64)), (256, 64, 4, 80 * 4 + 1, (TILE, 128), (TILE, 128)),
    (256, 192, 4, 48 * 4, (TILE, 128), (SKINNY, 64)), (256, 192, 4, 48 * 4 + 1, (TILE, 128), (TILE, 64)),
])
def test_down_tile(d, inter, active, rows, gu, dn):
    a, b = plan(layer(d, inter, active, 1), rows, active)
    assert ((a["kind"], a["bm"]), (b["kind"], b["bm"])) == (gu, dn), (a, b)


@pytest.mark.parametrize("rows,bm", [(1, 16), (16 * 8, 16), (16 * 8 + 1, 32), (32 * 8, 32), (32 * 8 + 1, 64), (9000, 64)])
def test_float32_tile_height(rows, bm):
    gu, dn = plan(layer(256, 512, 8, 2, dtype=X.F32), rows, 8)
    assert gu["kind"] == dn["kind"] == SIMT and gu["bm"] == dn["bm"] == bm
    assert gu["ksplit"] == dn["ksplit"] == 1  # the float32 kernel adds no partials


def test_query_validation():
    ly = layer(**MIXTRAL)
    out = (ctypes.c_int32 * 10)()
    L = X.lib()
    assert L.exfold_gemm_plan(ctypes.byref(ly), 64, 4, 256, None) == X.ERR_NULL
    assert L.exfold_gemm_plan(ctypes.byref(ly), -1, 4, 256, out) == X.ERR_SHAPE
    assert L.exfold_gemm_plan(ctypes.byref(ly), 64, 0, 256, out) == X.ERR_SHAPE
    assert L.exfold_gemm_plan(ctypes.byref(ly), 64, 4, 0, out) == X.ERR_SHAPE
    bad = layer(**MIXTRAL, dtype=7)
    assert L.exfold_gemm_plan(ctypes.byref(bad), 64, 4, 256, out) == X.ERR_DTYPE


def _tiles(p, sizes, out_cols, gate_up):
    """Tiles the device-side list holds for these group sizes under plan p."""
    n_tiles = out_cols // (p["bn"] // 2 if gate_up else p["bn"])
    if p["kind"] == WIDE:       # 128-row units, one tile per unit and pair of n-tiles
        return int(sum(-(-r // 128) for r in sizes)) * (n_tiles // 2)
    return int(sum(-(-r // p["bm"]) for r in sizes)) * n_tiles * p["ksplit"]


def _splits(rows, groups, rng):
    yield [rows] + [0] * (groups - 1)                     # one busy group
    q, r = divmod(rows, groups)
    yield [q + (i < r) for i in range(groups)]           # even
    if rows >= 129 * groups:                              # every group one row past a 128-row unit
        base = [128 * ((rows // groups - 1) // 128) + 1] * groups
        base[0] += rows - sum(base)
        yield base
    for _ in range(20):
        yield list(rng.multinomial(rows, rng.dirichlet(np.full(groups, 0.3))))


@pytest.mark.parametrize("shape,rows,active", [
    (MIXTRAL, 4096, 8), (MIXTRAL, 20000, 8), (MIXTRAL, 64, 4), (QWEN3, 32768, 128), (QWEN3, 1024, 16),
    (GLM, 4096 * 4 + 4096, 129), (GLM, 64 * 8 + 64, 33),
    (dict(d=384, inter=256, n=8, k=2), 8192, 8), (dict(d=2048, inter=1024, n=8, k=2), 9000, 8),
    (dict(d=1024, inter=2112, n=24, k=3), 400, 24), (dict(d=7168, inter=4160, n=8, k=2), 16, 2),
    (dict(d=256, inter=512, n=8, k=2, dtype=X.F32), 64, 8), (dict(d=640, inter=320, n=5, k=2, dtype=X.F32), 161, 5),
    (dict(d=128, inter=64, n=60, k=4, dtype=X.F32), 1200, 60),
])
def test_grids_cover_every_split(shape, rows, active):
    ly = layer(**shape)
    groups = shape["n"] + (1 if shape.get("shared") else 0)
    gu, dn = plan(ly, rows, active)
    rng = np.random.default_rng(rows)
    for sizes in _splits(rows, groups, rng):
        assert sum(sizes) == rows
        for p, cols, gate_up in ((gu, shape["inter"], True), (dn, shape["d"], False)):
            need = _tiles(p, sizes, cols, gate_up) + (256 if p["kind"] == WIDE else 0)
            assert p["grid"] >= need, (p, sizes)


# The calibration's pair sums hold a gate/up tile's rows in LDS, 128 at most: every plan stays within that, and
# the launch refuses a taller tile on the host.
def test_gate_up_tiles_fit_the_pair_sums():
    rng = np.random.default_rng(5)
    for _ in range(4000):
        d, inter, n = 128 * rng.integers(1, 65), 64 * rng.integers(1, 129), int(rng.integers(1, 257))
        ly = layer(int(d), int(inter), n, 1, dtype=X.F32 if rng.random() < 0.2 else X.BF16)
        gu, _ = plan(ly, int(np.exp(rng.uniform(0, np.log(1e6)))), n, int(rng.choice([64, 256, 304])))
        assert 1 <= gu["bm"] <= 128


@pytest.mark.skipif(torch.cuda.is_available(), reason="a host check: the call would launch if the check were missing")
@pytest.mark.parametrize("bm", [129, 256])
def test_pair_sums_refuse_a_taller_tile(bm):
    fn = getattr(X.lib(), "_ZN6exfold21launch_calib_finalizeEPKdPKsRKNS_11PermBuffersEiiiiddPdPfS8_S8_S7_P12ihipStream_t")
    i, f, v = ctypes.c_int, ctypes.c_double, ctypes.c_void_p
    fn.argtypes, fn.restype = [v, v, v, i, i, i, i, f, f, v, v, v, v, v, v], i
    buffers = (ctypes.c_void_p * 16)()
    assert fn(None, None, ctypes.addressof(buffers), bm, 4, 8, 2, 0.0, 0.0, *[None] * 6) == 1  # hipErrorInvalidValue
