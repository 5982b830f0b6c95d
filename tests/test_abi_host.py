"""Host-only checks of the C ABI: the library loads without a GPU, exports every symbol the
header declares, and rejects bad arguments before touching any memory."""
import ctypes as C
import os
import re

import pytest

from paper_2605_26632_amd import binding as rtl
from util import gemm_choice, row_split

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    hdr = open(os.path.join(ROOT, "include", "rtlynx.h")).read()
    declared = set(re.findall(r"\b(rtl_[a-z0-9_]+)\s*\(", hdr))
    assert declared == set(rtl.SYMBOLS), declared ^ set(rtl.SYMBOLS)
    L = rtl.lib()
    for name in declared:
        assert getattr(L, name) is not None
    assert rtl.version().startswith("rtlynx-gfx950")


def test_status_strings():
    for s in range(8):
        assert rtl.status_str(s).startswith("RTL_")
    assert rtl.status_str(7).startswith("RTL_ERR_ARCH") and rtl.status_str(99) == "RTL_ERR_UNKNOWN"


def test_init_reports_a_status_without_a_gpu():
    """rtl_init never aborts: without a usable device it reports RTL_ERR_HIP, on another AMD GPU
    RTL_ERR_ARCH, on a gfx950 device RTL_OK."""
    assert rtl.lib().rtl_init() in (0, 6, 7)


FAKE = 0x10000  # non-null, 256-byte aligned, never dereferenced: validation precedes any launch


def test_sparsify_pack_rejects_bad_arguments():
    L = rtl.lib()
    f = L.rtl_sparsify_pack
    ok_args = dict(X=FAKE, M=4, K=64, ldx=64, comp=1, eps=1e-8, vals=FAKE, meta=FAKE, scale=None,
                   ws=None, wsb=0, stream=None)

    def call(**kw):
        a = dict(ok_args, **kw)
        return f(a["X"], a["M"], a["K"], a["ldx"], a["comp"], a["eps"], a["vals"], a["meta"],
                 a["scale"], a["ws"], a["wsb"], a["stream"])

    assert call(K=12) == 2 and call(K=60) == 2          # K % 8
    assert call(ldx=32) == 2 and call(M=-1) == 2
    assert call(X=None) == 1 and call(vals=None) == 1 and call(meta=None) == 1
    assert call(comp=2) == 1 and call(comp=3) == 1       # ROW / TENSOR need `scale`
    assert call(X=FAKE + 2) == 3 and call(ldx=68) == 3
    assert call(comp=7) == 5 and call(eps=-1.0) == 5 and call(eps=float("nan")) == 5
    assert call(comp=3, scale=FAKE) == 4                 # TENSOR needs workspace
    assert call(comp=3, scale=FAKE, ws=FAKE, wsb=8) == 4
    assert call(M=0) == 0                                # empty input: OK, nothing launched
    assert L.rtl_sparsify_pack_workspace(100, 64, 3) == 800
    assert L.rtl_sparsify_pack_workspace(100, 64, 1) == 0


def test_linear_entry_points_reject_bad_arguments():
    L = rtl.lib()

    def dense(X=FAKE, W=FAKE, bias=None, Y=FAKE, M=4, N=4, K=64, ldx=64, ldw=64, ldy=4, ws=FAKE, wsb=1 << 30):
        return L.rtl_dense_linear(X, W, bias, Y, M, N, K, ldx, ldw, ldy, ws, wsb, None)

    def sparse(X=FAKE, W=FAKE, bias=None, Y=FAKE, M=4, N=4, K=64, ldx=64, ldw=64, ldy=4, comp=1,
               eps=1e-8, ws=FAKE, wsb=1 << 30):
        return L.rtl_sparse_linear(X, W, bias, Y, M, N, K, ldx, ldw, ldy, comp, eps, ws, wsb, None)

    for f in (dense, sparse):
        assert f(K=32) == 2 and f(K=0) == 2 and f(ldy=2) == 2 and f(ldw=32) == 2 and f(N=-3) == 2
        assert f(X=None) == 1 and f(W=None) == 1 and f(Y=None) == 1
        assert f(W=FAKE + 8) == 3 and f(ldx=68) == 3 and f(Y=FAKE + 1) == 3
        assert f(M=0) == 0 and f(N=0) == 0
    for f in (dense, sparse):        # more output tiles than a 32-bit grid index can number
        assert f(M=1 << 30, N=1 << 30, ldy=1 << 30) == 2
    for f in (dense, sparse):        # strides beyond the 32-bit tile-offset range are refused
        assert f(ldx=(1 << 22) + 8) == 2 and f(ldw=(1 << 22) + 8) == 2
    assert sparse(comp=9) == 5 and sparse(eps=float("inf")) == 5
    assert sparse(ws=None) == 4 and sparse(wsb=16) == 4 and sparse(ws=FAKE + 64) == 3
    need = L.rtl_sparse_linear_workspace(4096, 3072, 12288, 1)
    assert need >= 4096 * 12288 + 4096 * 12288 // 8

    def packed(vals=FAKE, meta=FAKE, W=FAKE, Y=FAKE, M=4, N=4, K=64, ldw=64, ldy=4):
        return L.rtl_packed_linear(vals, meta, None, None, W, None, Y, M, N, K, ldw, ldy, FAKE, 1 << 30, None)

    def lora(LA=FAKE, LB=FAKE, R=64, ldla=64, ldlb=64, ws=FAKE, wsb=1 << 30, K=64):
        return L.rtl_sparse_lora_linear(FAKE, FAKE, LA, LB, None, FAKE, 4, 4, K, R, K, K, ldla, ldlb, 4, 1, 1e-8,
                                        ws, wsb, None)

    assert lora(R=32) == 2 and lora(R=128) == 2 and lora(ldla=32) == 2 and lora(ldlb=32) == 2
    assert lora(LA=None) == 1 and lora(LB=None) == 1 and lora(LA=FAKE + 8) == 3 and lora(wsb=64) == 4
    assert L.rtl_sparse_lora_linear_workspace(4096, 3072, 12288, 64, 1) > L.rtl_sparse_linear_workspace(4096, 3072, 12288, 1)
    assert L.rtl_sparse_lora_linear_workspace(4096, 3072, 12288, 32, 1) == 0

    assert packed(meta=None) == 1 and packed(vals=None) == 1 and packed(K=96) == 2
    assert packed(meta=FAKE + 4) == 3 and packed(M=0) == 0


def test_fp8_entry_points_reject_bad_arguments():
    L = rtl.lib()

    def quant(W=FAKE, rows=4, cols=64, ld=64, Wq=FAKE, ldq=64):
        return L.rtl_quantize_fp8(W, rows, cols, ld, Wq, ldq, None)

    assert quant(cols=12) == 2 and quant(ld=32) == 2 and quant(ldq=32) == 2 and quant(rows=-1) == 2
    assert quant(W=None) == 1 and quant(Wq=None) == 1
    assert quant(W=FAKE + 2) == 3 and quant(Wq=FAKE + 4) == 3 and quant(ld=68) == 3
    assert quant(rows=0) == 0

    def pack(X=FAKE, M=4, K=64, ldx=64, comp=1, eps=1e-8, xs=FAKE, vals=FAKE, meta=FAKE, scale=None,
             ws=None, wsb=0):
        return L.rtl_sparsify_pack_fp8(X, M, K, ldx, comp, eps, xs, vals, meta, scale, ws, wsb, None)

    assert pack(K=12) == 2 and pack(ldx=32) == 2
    assert pack(xs=None) == 1 and pack(vals=None) == 1 and pack(comp=2) == 1
    assert pack(vals=FAKE + 2) == 3 and pack(xs=FAKE + 2) == 3
    assert pack(comp=5) == 5 and pack(eps=-1.0) == 5
    assert pack(comp=3, scale=FAKE) == 4
    assert pack(M=0) == 0

    def lin(X=FAKE, Wq=FAKE, xs=FAKE, Y=FAKE, M=4, N=4, K=128, ldx=128, ldw=128, ldy=4, comp=1, eps=1e-8,
            ws=FAKE, wsb=1 << 30):
        return L.rtl_sparse_linear_fp8(X, Wq, xs, None, Y, M, N, K, ldx, ldw, ldy, comp, eps, ws, wsb, None)

    assert lin(K=64, ldx=64, ldw=64) == 2 and lin(ldw=64) == 2 and lin(ldy=2) == 2
    assert lin(X=None) == 1 and lin(Wq=None) == 1 and lin(xs=None) == 1
    assert lin(ldw=136) == 3 and lin(Wq=FAKE + 8) == 3
    assert lin(comp=4) == 5
    assert lin(ws=None) == 4 and lin(wsb=8) == 4
    assert lin(M=0) == 0
    # half the value bytes of the bf16 workspace, same metadata
    assert L.rtl_sparse_linear_fp8_workspace(4096, 3072, 12288, 1) < L.rtl_sparse_linear_workspace(4096, 3072, 12288, 1)

    def lora(X=FAKE, Wq=FAKE, xs=FAKE, LA=FAKE, LB=FAKE, Y=FAKE, M=4, N=8, K=128, R=64, ldx=128, ldw=128, ldla=64,
             ldlb=128, ldy=8, comp=1, eps=1e-8, ws=FAKE, wsb=1 << 30):
        return L.rtl_sparse_lora_linear_fp8(X, Wq, xs, LA, LB, None, Y, M, N, K, R, ldx, ldw, ldla, ldlb, ldy, comp,
                                            eps, ws, wsb, None)

    assert lora(R=32) == 2 and lora(ldla=32) == 2 and lora(ldlb=64) == 2 and lora(K=64, ldx=64, ldw=64, ldlb=64) == 2
    assert lora(X=None) == 1 and lora(xs=None) == 1 and lora(LA=None) == 1 and lora(LB=None) == 1
    assert lora(LA=FAKE + 8) == 3 and lora(ldla=68) == 3 and lora(ldw=136) == 3 and lora(xs=FAKE + 2) == 3
    assert lora(comp=7) == 5 and lora(eps=float("nan")) == 5
    assert lora(ws=None) == 4 and lora(wsb=64) == 4
    assert lora(M=0) == 0 and lora(N=0) == 0
    need = L.rtl_sparse_lora_linear_fp8_workspace(4096, 3072, 12288, 64, 1)
    assert need > L.rtl_sparse_linear_fp8_workspace(4096, 3072, 12288, 1)       # + T planes + sweep scratch
    assert L.rtl_sparse_lora_linear_fp8_workspace(4096, 3072, 12288, 32, 1) == 0  # rank other than 64


def test_tile_plan_covers_the_output_exactly():
    """Host arithmetic of the launch plan: body tiles (256 x 256 or 256 x 192) on the first rows, 256 x 128
    tail tiles on the rest; together they cover every output element once, for any shape."""
    import random
    rnd = random.Random(5)
    shapes = [(4096, 3072), (4608, 12288), (16896, 3072), (1, 1), (255, 129), (257, 193), (100003, 40), (40, 70001)]
    shapes += [(rnd.randint(1, 20000), rnd.randint(1, 20000)) for _ in range(200)]
    for M, N in shapes:
        for dense in (False, True):
            p = rtl.diag_tile_plan(M, N, dense)
            assert p["body_width"] in (192, 256)
            tm = (M + 255) // 256
            rows = p["body_rows"]
            assert 0 <= rows <= M and (rows % 256 == 0 or rows == M)
            body_panels = (rows + 255) // 256
            assert p["body_tiles"] == body_panels * ((N + p["body_width"] - 1) // p["body_width"])
            assert p["tail_tiles"] == (tm - body_panels) * ((N + 127) // 128)
            assert p["body_tiles"] + p["tail_tiles"] >= 1
            if p["tail_tiles"] == 0:
                assert rows == M
    assert rtl.lib().rtl_diag_tile_plan(0, 5, 0, None) == 2 and rtl.lib().rtl_diag_tile_plan(5, 5, 0, None) == 1
    # the headline shape keeps its one-round plan: 256 tiles of 256 x 192, no tail
    assert rtl.diag_tile_plan(4096, 3072) == dict(body_width=192, body_rows=4096, body_tiles=256, tail_tiles=0)


def split_planes(query, M, N, K, *rest):
    """Bytes of partial planes in a linear's queried workspace: at N = 2^20 no contraction is split, so that query
    is the mandatory part alone."""
    return int(query(M, N, K, *rest)) - int(query(M, 1 << 20, K, *rest))


# The first five only split with fewer parts than the preferred number, because the room ends before: by 64 MiB in all
# for the entry point on the fixed scratch, whatever the other entry points' own mandatory part leaves.
SPLIT_SHAPES = [(2304, 1024, 15360), (2816, 512, 12288), (2304, 512, 15360), (1792, 1536, 18432), (2752, 512, 12288),
                (200, 3072, 12288), (333, 3072, 12288), (700, 3071, 12352), (140, 5504, 15360)]


def test_every_entry_point_plans_the_same_contraction_split():
    """The queries of all sparse entry points of an operand type ask for the same partial planes in every scope, and
    for planes wherever the entry point on the fixed scratch, which hands over all it has left, would split."""
    L = rtl.lib()
    limit = rtl.STATIC_SCRATCH_BYTES
    grid = [(M, N, K) for M in range(64, 4097, 448) for N in (256, 640, 1024, 2100, 3072, 5504) for K in (4096, 9216, 12288, 15360)]
    for M, N, K in SPLIT_SHAPES + [(3008, 1024, 12288), (2752, 1280, 12288)] + grid:
        planes = {split_planes(L.rtl_packed_linear_workspace, M, N, K)}
        fp8 = set()
        for comp in range(4):
            planes.add(split_planes(L.rtl_sparse_linear_workspace, M, N, K, comp))
            planes.add(split_planes(L.rtl_sparse_lora_linear_workspace, M, N, K, 64, comp))
            if L.rtl_sparse_linear_workspace(M, 1 << 20, K, comp) <= limit:
                assert L.rtl_sparse_linear_workspace(M, N, K, comp) <= limit      # what the fixed scratch takes
            if K % 128 == 0:
                fp8.add(split_planes(L.rtl_sparse_linear_fp8_workspace, M, N, K, comp))
                fp8.add(split_planes(L.rtl_sparse_lora_linear_fp8_workspace, M, N, K, 64, comp))
        assert len(planes) == 1 and len(fp8) <= 1, (M, N, K, planes, fp8)
        for p in planes | fp8:
            assert p == 0 or (p >= 2 * M * N * 4 and p % (M * ((N + 7) // 8 * 8) * 4) == 0)
        if (M, N, K) in SPLIT_SHAPES:
            assert min(planes) > 0, (M, N, K)


# Measured GPU time of a call, 256-row plan against the small tiles in several passes (us): the latter is the slower one.
@pytest.mark.parametrize("sparse,fp8,M,N,K", [
    (True, False, 1408, 14368, 11904),       # 303 / 392
    (True, False, 639, 10400, 11776),        # 137 / 169 (LoRA)
    (True, False, 1297, 5728, 5312),         # 59 / 64
    (True, False, 831, 17124, 6144),         # 145 / 149
    (True, False, 4973, 800, 4352),          # 59 / 71 (LoRA); 256 x 96 tiles in one pass 55
    (True, True, 858, 9024, 14592),          # 86 / 91
    (False, False, 4535, 4320, 13952),       # 481 / 581
    (False, False, 3960, 2036, 4096),        # 74 / 87
    (False, False, 884, 17575, 3840),        # 152 / 159
])
def test_tile_choice_keeps_the_256_row_plan_where_small_tiles_are_slower(sparse, fp8, M, N, K):
    """(or takes 256 x 96 tiles, which run in one pass only)"""
    assert gemm_choice(sparse, fp8, M, N, K)[:2] in ((-1, 1), (5, 1))


def test_tile_choice_where_small_tiles_are_faster():
    """[37, 3072, 12288] 69 us with the 256-row plan, 17 with 32 x 32 tiles in one pass; dense 125 and 20;
    [10, 16416, 11776] 32 x 32 tiles in three passes (all of W once) 1.27 times as fast as 128 x 128."""
    assert gemm_choice(True, False, 37, 3072, 12288) == (0, 1, 128)
    assert gemm_choice(True, False, 10, 16416, 11776)[:2] == (0, 1)
    assert gemm_choice(False, False, 37, 3072, 12288)[:2] != (-1, 1)
    assert gemm_choice(False, False, 333, 3072, 12288)[1] > 1
    for s in ((161, 6168, 128), (1981, 1024, 128), (2686, 640, 128), (319, 6336, 128)):      # dense 64 x 64: slower than the 256-row plan
        assert gemm_choice(False, False, *s)[0] in (3, 4)


def test_small_tile_shapes_of_the_gpu_tests_reach_every_tile():
    """The lists the parity tests run: every shape of the small-tile tables, sparse, dense and FP8, and the several-pass forms."""
    from test_parity_gpu import SMALL_TILE_SHAPES, SMALL_TILE_SHAPES_FP8
    for sparse, fp8, shapes in ((True, False, SMALL_TILE_SHAPES), (False, False, SMALL_TILE_SHAPES), (True, True, SMALL_TILE_SHAPES_FP8)):
        assert {gemm_choice(sparse, fp8, *s)[0] for s in shapes} >= set(range(6)), (sparse, fp8)
    assert gemm_choice(True, False, 1, 16421, 6144)[:2] == (0, 1)           # 514 tiles
    assert gemm_choice(False, False, 357, 21102, 1536)[:2] == (4, 1)        # 495 tiles


def test_waves_of_a_row_make_no_extra_trips():
    """The runs of a row's waves cover it once, in whole 512-element steps, and cost no more unrolled trips (1536 elements,
    paid in full when part of one lies past the run) than one wave alone; where the waves' sums meet in LDS their number
    divides the eight waves of a workgroup."""
    for comp in range(4):
        for M in (1, 37, 256, 300, 1024, 1025, 1500, 1537, 4608, 16896):
            for K in [8, 512, 1536, 1544] + list(range(2048, 20000, 520)) + [12288, 15360, 1 << 20]:
                parts, span = row_split(comp, M, K)
                assert 1 <= parts <= 8 and span % 512 == 0 and parts * span >= K
                runs = [max(0, min(K, (i + 1) * span) - i * span) for i in range(parts)]
                assert sum(runs) == K
                assert sum((r + 1535) // 1536 for r in runs) == (K + 1535) // 1536, (comp, M, K, parts, span)
                if comp >= 2:
                    assert 8 % parts == 0


@pytest.mark.parametrize("M,K,bf16_needs,fp8_needs", [(1, 128, False, False), (1024, 3072, False, False), (1025, 3072, True, True),
                                                      (1024, 3200, True, True), (1280, 1792, False, False), (1280, 2304, True, False),
                                                      (1281, 1792, True, True), (2048, 1536, False, False), (2049, 128, True, True)])
def test_lora_calls_without_k_ranges_ask_for_no_room_for_them(M, K, bf16_needs, fp8_needs):
    """Few rows with a short contraction have T = X L_B^T formed whole: operand and T are then all that a LoRA call needs."""
    L, N = rtl.lib(), 1 << 20                            # (no contraction is split at that width)
    t_bytes = (M * 64 * 4 + 255) // 256 * 256
    for needs, plain, lora, call in (
            (bf16_needs, L.rtl_sparse_linear_workspace, L.rtl_sparse_lora_linear_workspace,
             lambda n: L.rtl_sparse_lora_linear(FAKE, FAKE, FAKE, FAKE, 0, FAKE, M, N, K, 64, K, K, 64, K, N, 3, 1e-8, FAKE, n, 0)),
            (fp8_needs, L.rtl_sparse_linear_fp8_workspace, L.rtl_sparse_lora_linear_fp8_workspace,
             lambda n: L.rtl_sparse_lora_linear_fp8(FAKE, FAKE, FAKE, FAKE, FAKE, 0, FAKE, M, N, K, 64, K, K, 64, K, N, 3, 1e-8,
                                                    FAKE, n, 0))):
        whole = plain(M, N, K, 3) + t_bytes
        assert (lora(M, N, K, 64, 3) > whole) == needs
        assert call(whole - 1) == 4
        if needs:                                        # (an accepted call would launch where there is a device)
            assert call(whole) == 4


def test_kernels_need_no_scratch_memory(tmp_path):
    """No kernel of the library spills registers: scratch memory would cost every launch and is allocated by the runtime behind
    the caller's back. Read from the metadata notes of the code objects inside the built library."""
    import subprocess
    readelf = "/opt/rocm/llvm/bin/llvm-readelf"
    if not os.path.exists(readelf):
        pytest.skip("no llvm-readelf")
    blob = open(rtl.LIB_PATH, "rb").read()
    starts = [m.start() for m in re.finditer(b"\x7fELF\x02\x01\x01\x40", blob)]      # ELF64, OS ABI AMDGPU_HSA
    sizes, kernels = [], 0
    for n, at in enumerate(starts):
        p = tmp_path / ("%d.co" % n)
        p.write_bytes(blob[at:])
        notes = subprocess.run([readelf, "--notes", str(p)], capture_output=True, text=True).stdout
        kernels += notes.count(".symbol:")
        sizes += re.findall(r"\.private_segment_fixed_size:\s+(\d+)|\.vgpr_spill_count:\s+(\d+)", notes)
    assert kernels > 60
    assert {int(a or b) for a, b in sizes} == {0}
