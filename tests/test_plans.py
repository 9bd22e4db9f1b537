"""Launch shapes of the library's planners, read from the built library's own
planning functions (host code: no device is needed)."""
import ctypes as C

import pytest

from paper_1609_06119_amd._lib import LIB_PATH

CUS, LDS = 256, 160 * 1024          # compute units and LDS bytes of an MI355X
RESERVE = 1024                      # LDS kept aside for static arrays
SPLIT_EVENTS = 256                  # events of a few-events workgroup


class ApplyShape(C.Structure):
    _fields_ = [("shallow", C.c_bool), ("split", C.c_bool), ("table_far", C.c_bool),
                ("missing", C.c_bool), ("threads", C.c_int), ("blocks", C.c_int),
                ("trees_per_chunk", C.c_int), ("d_used", C.c_int), ("node_stride", C.c_int),
                ("lds_bytes", C.c_size_t)]


class IntVector(C.Structure):       # std::vector<int>: begin, end, end of storage
    _fields_ = [("begin", C.POINTER(C.c_int)), ("end", C.POINTER(C.c_int)), ("cap", C.c_void_p)]


@pytest.fixture(scope="module")
def planner():
    lib = C.CDLL(LIB_PATH)
    plan = getattr(lib, "_ZN4fbdt10plan_applyEliiibimim")
    plan.restype = ApplyShape
    plan.argtypes = [C.c_int64, C.c_int, C.c_int, C.c_int, C.c_bool, C.c_int, C.c_size_t, C.c_int,
                     C.c_size_t]
    strides = getattr(lib, "_ZN4fbdt18apply_node_stridesEiiibimim")
    strides.restype = IntVector
    strides.argtypes = plan.argtypes[1:]

    class Planner:
        def apply(self, n, d, T, D, missing=False, threads=0, table=0):
            return plan(n, d, T, D, missing, CUS, LDS, threads, table)

        def strides(self, d, T, D, missing=False, threads=0, table=0):
            v = strides(d, T, D, missing, CUS, LDS, threads, table)
            count = (C.cast(v.end, C.c_void_p).value - C.cast(v.begin, C.c_void_p).value) // 4
            return [v.begin[k] for k in range(count)]

    return Planner()


def tree_bytes(s, D):
    """LDS bytes of a tree: its boost weights, and the deep kernels' records."""
    nin = (1 << D) - 1
    return (2 * nin + 1 if s.missing else nin + 1) * 8 + (0 if s.shallow else nin * 4)


FORESTS = [(1, 1, False), (10, 1, False), (400, 3, False), (3000, 3, False), (100, 4, False),
           (100, 6, False), (1000, 7, False), (300, 2, True), (200, 7, True)]
WIDTHS = [1, 2, 5, 13, 40, 60, 79, 80, 100, 125, 142, 143, 150, 155, 156, 157, 158, 159, 160, 180,
          210, 211, 212, 254, 255]
EVENTS = [1, 255, 256, 257, 65_536, 393_216, 393_217, 600_000, 1_300_001, 50_000_000, 1 << 33]


def table_bytes(d, levels):
    """A float input's table with 2^levels words of thresholds per feature."""
    return 4 * d * (1 + (1 << levels))


@pytest.mark.parametrize("T,D,missing", FORESTS)
def test_apply_shapes_hold(planner, T, D, missing):
    """Every shape fits the LDS and the launch limits, covers its events, and
    has the node records that the model's first call makes."""
    for d in WIDTHS:
        for table in (0, table_bytes(d, 1), table_bytes(d, 5), table_bytes(d, 7), table_bytes(d, 8)):
            known = set(planner.strides(d, T, D, missing, 0, table))
            for n in EVENTS:
                s = planner.apply(n, d, T, D, missing, 0, table)
                what = (d, table, n)
                extra = 0 if s.table_far else (table + 15) // 16 * 16
                per = tree_bytes(s, D) + (SPLIT_EVENTS if s.split else 0)
                events = SPLIT_EVENTS if s.split else 4 * s.threads
                assert s.shallow == (D <= 3 and not missing), what
                assert s.threads % 64 == 0 and 64 <= s.threads <= 1024, what
                assert 1 <= s.trees_per_chunk <= T, what
                assert s.lds_bytes >= s.trees_per_chunk * per + d * events + extra, what
                assert s.lds_bytes + RESERVE <= LDS, what
                assert s.node_stride == events and s.node_stride in known, what
                assert s.blocks >= 1 and s.blocks * s.threads < 1 << 32, what
                if s.split:
                    assert s.blocks * SPLIT_EVENTS >= n, what
                assert table or not s.table_far, what


@pytest.mark.parametrize("T,D,missing", FORESTS)
def test_a_bulk_launch_fills_the_compute_units(planner, T, D, missing):
    """A bulk launch holds at least 8 wavefronts per compute unit: where the
    code tile of a wide forest or the threshold table of float values leaves
    room for fewer, the wavefronts of a few-events launch share the trees."""
    for d in range(1, 256):
        for levels in (0, 2, 5, 8):
            table = table_bytes(d, levels) if levels else 0
            for n in (393_217, 2_000_000, 50_000_000):
                s = planner.apply(n, d, T, D, missing, 0, table)
                per_cu = LDS // (s.lds_bytes + RESERVE)
                assert s.split or per_cu * s.threads >= 8 * 64, (d, levels, n, s.threads)


@pytest.mark.parametrize("T,D,missing", FORESTS + [(12_000, 3, False), (12_000, 2, False)])
def test_a_threshold_table_leaves_room_for_trees(planner, T, D, missing):
    """A few-events launch keeps the threshold table of float values in LDS
    only where that adds at most 16 chunks of trees to the launch."""
    near = 0
    for d in range(1, 256):
        plain = planner.apply(500, d, T, D, missing, 0, 0)
        assert plain.split
        for levels in range(1, 9):
            s = planner.apply(500, d, T, D, missing, 0, table_bytes(d, levels))
            what = (d, levels, s.trees_per_chunk)
            assert s.split, what
            if s.table_far:
                assert s.trees_per_chunk == plain.trees_per_chunk, what
            else:
                near += 1
                assert -(-T // s.trees_per_chunk) <= -(-T // plain.trees_per_chunk) + 16, what
    assert near > 0


class QuantileShape(C.Structure):
    _fields_ = [("small", C.c_bool), ("chunks", C.c_int), ("per", C.c_int64)]


@pytest.fixture(scope="module")
def quantile_plan():
    plan = C.CDLL(LIB_PATH)._ZN4fbdt14plan_quantilesElii
    plan.restype = QuantileShape
    plan.argtypes = [C.c_int64, C.c_int, C.c_int]
    return lambda n, d: plan(n, d, CUS)


def test_quantile_shapes_cover_their_values(quantile_plan):
    for d in (1, 2, 7, 8, 40, 100, 255):
        for n in (1, 20_480, 40_960, 40_961, 65_281, 300_001, 4_000_001, 50_000_000, 1 << 33):
            q = quantile_plan(n, d)
            assert q.small == (n <= 40_960), (n, d)
            if not q.small:
                assert 1 <= q.chunks <= 256 and q.per % 4 == 0, (n, d)
                assert (q.chunks - 1) * q.per < n <= q.chunks * q.per, (n, d)
                assert q.per <= 1 << 31, (n, d)


def test_the_swept_cases_sweep(quantile_plan):
    """The binning tests' cases of long chunks take the 32-bit counters, and
    one of them has a last chunk that needs none for itself."""
    from test_gpu_quantiles import SWEPT
    last = []
    for n, d, _, _ in SWEPT:
        q = quantile_plan(n, d)
        assert q.per > 65_280, (n, d)
        last.append(n - (q.chunks - 1) * q.per)
    assert min(last) <= 65_280


class HistShape(C.Structure):
    _fields_ = [("features_per_group", C.c_int), ("feature_groups", C.c_int),
                ("nodes_per_group", C.c_int), ("node_groups", C.c_int), ("chunks", C.c_int),
                ("chunk_events", C.c_int64), ("xcd_events", C.c_int64), ("threads", C.c_int),
                ("blocks", C.c_int), ("copies", C.c_int), ("copy_stride", C.c_int),
                ("lds_bytes", C.c_size_t), ("sibling", C.c_bool), ("prefix", C.c_bool)]


@pytest.mark.parametrize("n,d,n_bins,layer,shape", [
    (2_900_000, 40, 256, 0, (5, 32)), (200_000, 27, 200, 0, (1, 8)), (200_000, 27, 200, 1, (1, 8)),
    (500_000, 20, 256, 0, (2, 24)), (50_000, 100, 256, 4, (2, 8)), (1_000_000, 40, 64, 2, (5, 32)),
])
def test_a_histogram_by_itself_takes_few_chunks(n, d, n_bins, layer, shape):
    """fbdt_histogram's chunks are summed one after another by a pass of its
    own, so its shapes (features per group, chunks) are not those of a fit's
    layers; these were the fastest or within 4% of it when timed."""
    plan = C.CDLL(LIB_PATH)._ZN4fbdt14plan_histogramEliiibbimRKNS_13HistOverridesE
    plan.restype = HistShape
    plan.argtypes = [C.c_int64, C.c_int, C.c_int, C.c_int, C.c_bool, C.c_bool, C.c_int,
                     C.c_size_t, C.c_void_p]
    s = plan(n, d, n_bins, layer, False, False, CUS, LDS, C.byref((C.c_int * 4)()))
    assert (s.features_per_group, s.chunks) == shape
