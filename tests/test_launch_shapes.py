"""Launch shapes of the projections, asked of the library's own functions on the host: needs no GPU."""
import ctypes as C

import pytest

from paper_2501_08090_amd import binding as B

STEP, BLOCK, ALONE = range(3)  # SliceCost
MOST = 16                      # linear_max_split()


class Linear(C.Structure):
    _fields_ = [("w", C.c_void_p), ("N", C.c_int), ("K", C.c_int), ("Npad", C.c_int), ("Kpad", C.c_int), ("tstride", C.c_size_t), ("owned", C.c_bool)]


class Shape(C.Structure):
    _fields_ = [(n, C.c_int) for n in ("mt", "nf", "nw", "ks", "gx", "gz", "ksplit", "cps")]

    def key(self):
        """tile, K-slices and chunks per slice (eight waves of half the columns are four of whole ones)"""
        return self.mt, self.nf * self.nw // 4, self.ksplit, self.cps


def linear(N, K):
    return Linear(None, N, K, (N + 31) // 32 * 32, (K + 255) // 256 * 256, 0, False)


def shape(N, K, M, sliceable=True, slices=STEP, swept=False):
    f = B.load()._ZN6chiron12linear_shapeERKNS_6LinearEibiiNS_9SliceCostEb
    f.restype = Shape
    return f(C.byref(linear(N, K)), C.c_int(M), C.c_bool(sliceable), C.c_int(0), C.c_int(MOST if sliceable else 1), C.c_int(slices), C.c_bool(swept))


def searches():
    f = B.load()._ZN6chiron21linear_shape_searchesEv
    f.restype = C.POINTER(C.c_int64)
    return f()[0]


# QKV, O, gate/up, down and head: (N, K, sliceable)
def products(H, qkv, qn, F, vocab):
    return (qkv, H, True), (H, qn, True), (2 * F, H, False), (H, F, True), (vocab, H, False)


WIDTHS = {"8b": products(4096, 6144, 4096, 14336, 128256), "70b": products(8192, 10240, 8192, 28672, 128256)}


@pytest.mark.parametrize("widths", [WIDTHS["8b"], WIDTHS["70b"], products(5120, 7168, 5120, 13824, 32000), products(1024, 1536, 1024, 2816, 32768),
                                    products(256, 512, 256, 688, 1024)])
def test_a_step_searches_for_each_product_once(widths):
    """the five products of a step are asked for layer after layer: only the first layer, the head and another row count search"""
    for M in (64, 128, 500, 437):
        before = searches()
        for _ in range(3):
            for _ in range(32):
                for N, K, sliceable in widths[:4]:
                    shape(N, K, M, sliceable)
            shape(*widths[4][:2], M, widths[4][2])
        assert searches() - before <= 5


@pytest.mark.parametrize("M,N,K", [(128, 2048, 2048), (182, 4254, 3056), (157, 517, 7648), (325, 941, 1488), (163, 2091, 1968)])
@pytest.mark.parametrize("slices", [BLOCK, ALONE])
def test_sliced_shapes_are_compared_by_their_kernels(M, N, K, slices):
    """what a call with slices takes at least is no reason to take a slower sliced shape: the shape is the one inside a step, where
    there is no such floor"""
    assert shape(N, K, M, slices=STEP).ksplit > 1
    assert shape(N, K, M, slices=slices).key() == shape(N, K, M, slices=STEP).key()


# where the estimate replaces the shape of the rules at the widths that those were swept at, up to 256 rows (the comment at the
# estimate has the times of both): {(widths, product of `products`): rows}
REPLACED = {("8b", 0): [*range(65, 97)], ("8b", 1): [*range(65, 97), *range(129, 193)], ("8b", 4): [96],
            ("70b", 0): [*range(129, 193)], ("70b", 3): [*range(129, 153), *range(193, 224)], ("70b", 4): [96]}


@pytest.mark.parametrize("widths", WIDTHS)
def test_the_swept_widths_keep_the_shapes_that_were_swept(widths):
    """up to 256 rows every launch at the 8B and 70B widths has the shape of the rules, but for those that were timed with the other;
    no slice gets longer than 1024 inputs, or the rules' own, by it"""
    for i, (N, K, sliceable) in enumerate(WIDTHS[widths]):
        other = [M for M in range(1, 257) if shape(N, K, M, sliceable).key() != shape(N, K, M, sliceable, swept=True).key()]
        assert other == REPLACED.get((widths, i), []), (N, K)
        assert all(shape(N, K, M).cps <= max(16, shape(N, K, M, swept=True).cps) for M in other if sliceable)


def test_a_forced_start_of_the_two_term_form_ends_the_few_rows():
    """linear_big_min_m at 17 .. 32 rows takes effect where the few-row kernel would pay; up to 16 rows that kernel comes first, as ever"""
    f = B.load()._ZN6chiron15linear_few_rowsEi
    f.restype = C.c_bool
    few = lambda M: f(C.c_int(M))
    assert [few(M) for M in (1, 16, 17, 32, 33)] == [True, True, True, True, False]
    try:
        for start, want in ((1, [True, False, False, False]), (20, [True, True, False, False]), (33, [True] * 4), (-1, [True] * 4)):
            B.set_tuning("linear_big_min_m", start)
            assert [few(M) for M in (16, 19, 20, 32)] == want, start
    finally:
        B.set_tuning("linear_big_min_m", 0)


# hidden, QKV, O's inputs, ffn: {rows: us per layer that a step gains by the few-row kernels, measured end to end}
GAINED = {(4096, 6144, 4096, 14336): {1: 9, 8: 6, 12: 1, 16: -4}, (8192, 10240, 8192, 28672): {1: 6, 9: 6, 10: 5, 11: 2, 16: -9},
          (4096, 12288, 4096, 11008): {1: 6, 8: 5, 11: 2, 16: -4}, (2048, 10240, 8192, 8192): {1: 5, 4: 4, 8: 1},
          (5120, 15360, 5120, 13824): {1: 5, 4: 3, 8: -4, 11: -10}, (5120, 12288, 8192, 13824): {8: -6, 11: -12}, (4608, 13824, 4608, 12288): {8: -6, 11: -9},
          (7168, 10240, 8192, 20480): {1: 5, 4: 4, 7: 3, 11: -8}, (3584, 10240, 8192, 9728): {1: 5, 4: 4, 6: 4}, (3072, 10240, 8192, 8192): {1: 5, 4: 4, 10: -4},
          (2560, 10240, 8192, 8192): {8: -6, 10: -7}, (6144, 18432, 6144, 16384): {1: 10, 8: 6, 11: -4}, (5120, 6144, 4096, 13824): {1: 8, 10: 2, 16: -8},
          (6144, 6144, 4096, 16384): {1: 16, 14: 6}, (4608, 6144, 4096, 8192): {1: 17, 11: 6}}


@pytest.mark.parametrize("widths", GAINED)
def test_a_step_takes_the_few_row_kernels_where_they_gained(widths):
    H, qkv, qn, F = widths
    f = B.load()._ZN6chiron13step_few_rowsERKNS_6LinearES2_S2_S2_i
    f.restype = C.c_bool
    ops = [linear(qkv, H), linear(H, qn), linear(2 * F, H), linear(H, F)]
    for M, gain in GAINED[widths].items():
        assert f(*(C.byref(o) for o in ops), C.c_int(M)) == (gain > 0), (widths, M)
