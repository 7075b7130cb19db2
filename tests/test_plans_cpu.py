"""Which kernel a call runs on and how its launch is cut: the planners are host
functions of libjf (paper_2512_14681_amd/csrc/jf_internal.h), called here by
their C++ names, without a GPU."""
import ctypes
import glob
import os
import re

import pytest

from paper_2512_14681_amd import jf

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2512_14681_amd", "csrc")
I = ctypes.c_int
(SEL_GENERAL, SEL_MULTI_5, SEL_MULTI_8, SEL_MULTI_17, SEL_WIDE_16, SEL_WIDE_32_1, SEL_WIDE_32_3,
 SEL_WIDE_32_4) = range(8)


@pytest.fixture(scope="module")
def L():
    if not os.path.exists(jf.LIB_PATH):
        pytest.skip("libjf.so not built (python -m paper_2512_14681_amd.build)")
    return ctypes.CDLL(jf.LIB_PATH)


# ---- many-row GEMM ------------------------------------------------------------------
EPI_STORE, EPI_RESID, EPI_QKV, EPI_SWIGLU, EPI_ARGMAX = range(5)
CUS = 256


class MrPlan(ctypes.Structure):
    _fields_ = [(k, I) for k in ("R", "RT", "CT", "KC", "P", "T", "gr", "n_cg", "S", "chunks", "any")]


def mr_plan(L, R, N, K, epi, splits=64, aligned=True):
    """The many-row GEMM's plan of [R][K] x [N][K]^T, or None: another kernel runs it."""
    f = L._ZN2jf12gemm_mr_planERNS_6MrPlanEiiiiiib
    f.restype, f.argtypes = ctypes.c_bool, [ctypes.POINTER(MrPlan), I, I, I, I, I, I, ctypes.c_bool]
    m = MrPlan()
    return m if f(ctypes.byref(m), R, N, K, epi, CUS, splits, aligned) else None


# An LM head (rows, words, width; no split-K scratch) for every block shape of
# the many-row kernel that such a call reaches, {(RT, CT): (R, V, d)}: RT row
# tiles by CT column tiles.  The last row tile of the last chunk is there and
# ragged; 16 stages, more than any ring is deep, but where V is small.
MANY_ROW_BLOCKS = {
    (2, 8): (17, 32768, 512), (2, 12): (17, 32784, 512), (4, 2): (246, 1600, 512), (4, 4): (113, 4112, 512),
    (4, 6): (241, 4112, 512), (4, 8): (241, 6400, 512), (4, 10): (241, 8208, 512), (4, 12): (113, 22400, 512),
    (6, 4): (177, 2560, 512), (6, 8): (369, 4112, 512), (6, 12): (177, 16400, 512), (8, 2): (497, 1024, 512),
    (8, 4): (497, 2560, 512), (8, 6): (497, 4112, 512), (8, 8): (497, 6400, 512), (8, 10): (497, 8208, 512),
    (8, 12): (497, 11200, 512), (10, 4): (305, 4112, 512), (10, 8): (305, 8208, 512), (10, 12): (305, 16400, 512),
    (10, 16): (305, 24592, 512), (12, 2): (369, 1344, 128), (12, 4): (369, 7232, 256), (12, 6): (369, 8208, 512),
    (12, 8): (369, 12304, 512), (12, 10): (369, 16400, 512), (12, 12): (369, 22400, 512), (16, 2): (497, 3136, 128),
    (16, 4): (497, 6208, 128), (16, 6): (497, 12288, 512), (16, 8): (497, 12304, 512), (16, 10): (497, 16400, 512)}

# The same for operands off a 16-byte boundary.
ANY_ALIGNMENT_BLOCKS = {
    (4, 2): (246, 1600, 512), (4, 4): (113, 4112, 640), (4, 6): (241, 4112, 512), (4, 8): (49, 27200, 640),
    (4, 10): (113, 16400, 512), (4, 12): (49, 40976, 512), (6, 4): (369, 1600, 512), (6, 8): (369, 4112, 512),
    (6, 12): (369, 8208, 512), (8, 2): (497, 1024, 512), (8, 4): (497, 2560, 512), (8, 6): (497, 4112, 512),
    (8, 8): (497, 6400, 512), (8, 10): (497, 8208, 512), (8, 12): (497, 11200, 512)}


def instantiated_blocks(files):
    """(RT, CT) of every k_gemm_mr in the sources that match `files`."""
    out = set()
    for path in glob.glob(os.path.join(CSRC, files)):
        with open(path) as f:
            for mt, nt, wm, wn in re.findall(r"return launch_mr_cfg<(\d+), (\d+), (\d+), (\d+),", f.read()):
                out.add((int(mt) * int(wm), int(nt) * int(wn)))
    return out


@pytest.mark.parametrize("aligned", [True, False])
def test_every_block_shape_has_a_case(L, aligned):
    """The cases run on the block shapes they are listed under, and are all
    there are, but for the one that only split K reaches: a down projection's
    at 25 to 32 rows (the 32-row step of the mid-size decoder)."""
    cases = MANY_ROW_BLOCKS if aligned else ANY_ALIGNMENT_BLOCKS
    for (rt, ct), (R, V, d) in cases.items():
        m = mr_plan(L, R, V, d, EPI_ARGMAX, splits=1, aligned=aligned)
        assert m and (m.RT, m.CT, m.S) == (rt, ct, 1), ((rt, ct), m and (m.RT, m.CT, m.S))
        last = R - (m.chunks - 1) * 16 * rt
        assert 16 * (rt - 1) < last < 16 * rt
    if aligned:
        down = mr_plan(L, 32, 2048, 8192, EPI_RESID)
        assert (down.RT, down.CT) == (2, 4) and down.S > 1
        assert set(cases) | {(2, 4)} == instantiated_blocks("gemm_mr_rt*.hip")
    else:
        assert set(cases) == instantiated_blocks("gemm_mr_any.hip")


@pytest.mark.parametrize("R,N,K", [(320, 4608, 2560), (448, 4608, 2560), (160, 6144, 2560), (320, 6144, 2560),
                                   (320, 3072, 2048), (448, 3072, 2048), (448, 1280, 1024), (512, 4608, 3584),
                                   (512, 6144, 4096)])
def test_qkv_splits_k_where_its_epilogue_would_stall(L, R, N, K):
    """The QKV epilogue of a workgroup without split K takes longer than the
    split and its reduction (us, one split -> these plans, in this order: 41.6
    -> 32.0, 44.9 -> 35.9, 31.7 -> 29.2, 43.5 -> 36.1, 27.9 -> 24.7, 31.7 ->
    25.9, 18.0 -> 15.4, 52.1 -> 45.5, 64.4 -> 55.9)."""
    assert mr_plan(L, R, N, K, EPI_QKV).S > 1


def test_long_k_stays_on_the_many_row_kernel(L):
    """A long-K down projection, however narrow, is on the many-row kernel at
    every row count from 17 on (its bound once left 33 to 64 rows out)."""
    for N in (512, 1024, 1536, 1920, 2560, 3072, 3328, 3840, 4096):
        for R in range(17, 129):
            assert mr_plan(L, R, N, 8192, EPI_RESID), (R, N)
            assert mr_plan(L, R, N, 18944, EPI_RESID), (R, N)


@pytest.mark.parametrize("N,K,epi,here", [
    (4096, 4096, EPI_RESID, False), (4096, 6144, EPI_RESID, False), (3712, 5120, EPI_RESID, False),
    (4096, 7552, EPI_RESID, True), (2560, 6912, EPI_RESID, True), (3072, 5504, EPI_RESID, True),
    (3584, 3584, EPI_RESID, False), (8192, 2048, EPI_ARGMAX, False), (8192, 3584, EPI_ARGMAX, True),
    (8208, 2048, EPI_ARGMAX, True), (4608, 3584, EPI_QKV, True), (4352, 4096, EPI_QKV, True),
    (6144, 4096, EPI_QKV, True),
    (16384, 2048, EPI_SWIGLU, True), (37888, 3584, EPI_SWIGLU, True),
    (16384, 1024, EPI_SWIGLU, True), (32000, 512, EPI_ARGMAX, True)])
def test_33_to_64_rows_by_what_the_streaming_kernel_fills(L, N, K, epi, here):
    """Matrices of at most two column tiles a unit whose two row chunks make one
    full round of the weight-streaming kernel's waves stay on it up to 26M
    elements."""
    for R in (33, 48, 64):
        assert (mr_plan(L, R, N, K, epi) is not None) == here


def test_the_few_row_step_of_the_wide_decoder(L):
    """The decoder of the GPU parity test at 10 to 16 rows has its gate/up
    projection here."""
    for R in (10, 13, 15, 16):
        m = mr_plan(L, R, 2 * 20480, 256, EPI_SWIGLU)
        assert m and m.RT == 2 and m.chunks == 1


@pytest.mark.parametrize("N,K,epi,splits,here", [
    (37888, 3584, EPI_SWIGLU, 64, True), (40960, 512, EPI_SWIGLU, 64, True), (49152, 1024, EPI_SWIGLU, 64, False),
    (32768, 3072, EPI_SWIGLU, 64, False), (28672, 4096, EPI_SWIGLU, 64, False), (49152, 256, EPI_ARGMAX, 64, True),
    (49152, 256, EPI_ARGMAX, 1, False), (40960, 2048, EPI_ARGMAX, 1, True), (152064, 3584, EPI_ARGMAX, 64, False),
    (32768, 8192, EPI_ARGMAX, 1, True)])
def test_10_to_16_rows_where_the_streaming_rounds_are_uneven(L, N, K, epi, splits, here):
    """Few rows go to the many-row kernel where one round of its workgroups
    holds the matrix and the weight-streaming kernel's last round is partly
    empty, for a step's LM head of that width, and for very large ones."""
    for R in (1, 8, 9):
        assert mr_plan(L, R, N, K, epi, splits) is None
    for R in (10, 13, 16):
        assert (mr_plan(L, R, N, K, epi, splits) is not None) == here


@pytest.mark.parametrize("R,N,K,here", [
    (17, 1024, 8192, False), (24, 8192, 8192, False), (32, 4096, 8192, False), (17, 16384, 8192, False),
    (17, 32768, 8192, True), (32, 32768, 8192, True), (33, 8192, 2048, False), (40, 8192, 5120, False),
    (33, 12288, 3584, True), (64, 16384, 8192, True), (192, 2048, 3584, False), (256, 2048, 3584, True),
    (320, 1024, 3584, False), (448, 1024, 8192, False), (448, 2048, 8192, False), (65, 4096, 8192, True),
    (65, 8192, 1024, True)])
def test_lm_head_without_split_k_scratch(L, R, N, K, here):
    """The LM-head component has no scratch for split K: narrow heads and long
    K stay on the weight-streaming kernel, whose waves share K; with the
    scratch long K is on the many-row kernel."""
    m = mr_plan(L, R, N, K, EPI_ARGMAX, splits=1)
    assert (m is not None) == here
    assert m is None or m.S == 1
    if K >= 8192 and R >= 25:
        assert mr_plan(L, R, N, K, EPI_ARGMAX) is not None


def test_operands_off_a_16_byte_boundary(L):
    """They have the many-row kernel too, from 33 rows, in the chunks that are
    built for them and for the same matrices."""
    for N, K, epi in ((37888, 3584, EPI_SWIGLU), (3584, 18944, EPI_RESID), (4608, 3584, EPI_QKV),
                      (3584, 3584, EPI_RESID), (8192, 3584, EPI_ARGMAX), (1024, 1024, EPI_RESID)):
        for R in list(range(1, 129)) + [192, 320, 512]:
            m, a = mr_plan(L, R, N, K, epi, aligned=False), mr_plan(L, R, N, K, epi)
            assert a is None or a.any == 0
            if R < 33:
                assert m is None
            else:
                assert (m is None) == (a is None)
                assert m is None or (m.any == 1 and (m.RT, m.CT) in ANY_ALIGNMENT_BLOCKS)


# ---- trajectory selection ---------------------------------------------------------
def select_form(L, n, max_points, w=16, counts=False):
    f = L._ZN2jf16traj_select_formEiiib
    f.restype, f.argtypes = I, [I, I, I, ctypes.c_bool]
    return f(n, max_points, w, counts)


def test_selection_loads_match_the_points(L):
    """No more loads than the points need (the kernel runs one for points
    that are not there as well), and no fewer: 64 lanes load PP = 16 (n = 16)
    or 8 (n = 32) points before the fixed point each time."""
    for P in range(2, 70):
        f16, f32 = select_form(L, 16, P), select_form(L, 32, P)
        assert (f16 == SEL_WIDE_16) == (P - 1 <= 16)
        loads = {SEL_WIDE_32_1: 1, SEL_WIDE_32_3: 3, SEL_WIDE_32_4: 4}.get(f32)
        if loads:
            need = (P - 1 + 7) // 8
            assert need <= loads <= need + (P == 17)
        else:
            assert 10 <= P <= 16 or P > 33
    assert select_form(L, 16, 1) == SEL_MULTI_5 and select_form(L, 32, 1) == SEL_MULTI_5


@pytest.mark.parametrize("n,P,w,form", [
    (8, 9, 16, SEL_MULTI_5), (24, 25, 16, SEL_MULTI_17), (32, 13, 16, SEL_MULTI_8), (32, 40, 16, SEL_GENERAL),
    (65, 5, 16, SEL_GENERAL), (16, 65, 16, SEL_GENERAL), (16, 9, 1 << 24, SEL_GENERAL),
    (16, 9, 1 << 21, SEL_GENERAL)])
def test_selection_general_forms(L, n, P, w, form):
    assert select_form(L, n, P, w) == form


def test_selection_with_counts_keeps_one_store_a_block(L):
    for n, P in ((16, 17), (32, 5), (32, 33)):
        assert select_form(L, n, P, counts=True) < SEL_WIDE_16
