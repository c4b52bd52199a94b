"""What the built kernels take of a CU, read from the metadata of the library's own
code objects, and the launch plans that count on it (CPU only)."""
import ctypes
import random
import re

import pytest

from paper_2606_03928_amd import vase

KIND = {0: "pass1", 1: "pass2", 2: "fused"}
LDS, LDS_STEP = 160 * 1024, 1280


def _kernels():
    msgpack = pytest.importorskip("msgpack")
    with open(vase.LIB_PATH, "rb") as f:
        blob = f.read()
    out, at = {}, blob.find(b"\xaeamdhsa.kernels")
    while at >= 0:
        u = msgpack.Unpacker(raw=False, strict_map_key=False)
        u.feed(blob[at - 1:at + (8 << 20)])          # the map's head is the byte before its first key
        out.update((k[".name"], k) for k in u.unpack()["amdhsa.kernels"])
        at = blob.find(b"\xaeamdhsa.kernels", at + 1)
    assert out
    return out


@pytest.fixture(scope="module")
def kernels():
    vase.load()
    return _kernels()


def _score_kernels(kernels):
    """(d, waves, pass) -> the instantiations of the bf16 score kernel."""
    out = {}
    for name, k in kernels.items():
        m = re.search(r"score_mfma_kernelILi(\d+)ELi(\d+)ELi(\d)ELi(\d)ELb(\d)E", name)
        if m:
            out.setdefault((int(m[1]), int(m[2]), KIND[int(m[3])]), []).append(k)
    assert len(out) == 12
    return out


def test_no_kernel_spills_registers(kernels):
    assert not {n: k[".vgpr_spill_count"] for n, k in kernels.items() if k[".vgpr_spill_count"]}


def test_score_kernels_take_what_the_plan_counts(kernels):
    for (d, waves, kind), ks in _score_kernels(kernels).items():
        lds = 8 * 32 * d * 2 + 256 + (waves * 256 if kind != "pass2" else 0) + (
            waves * 512 if kind != "pass1" else 0)
        # workgroups of four waves that the registers leave to a CU
        most = 3 if (d, kind) == (64, "pass2") else 2
        for k in ks:
            assert k[".group_segment_fixed_size"] <= lds
            assert (k[".vgpr_count"] + k[".agpr_count"] + 7) // 8 * 8 * most <= 512


class Plan(ctypes.Structure):
    _fields_ = ([(n, ctypes.c_int) for n in ("n_chunk1", "n_chunk2", "n_slab", "rows_per_slab",
                                             "waves", "split_keys")] +
                [("mfma", ctypes.c_bool), ("pool_in_kernel", ctypes.c_bool)] +
                [(n, ctypes.c_size_t) for n in ("off_part", "off_col", "bytes")])


def _score_plan():
    f = vase.load()["_ZN4vase10score_planEiiiiiiib"]   # vase::score_plan of vase_internal.hpp
    f.restype = Plan
    f.argtypes = [ctypes.c_int] * 7 + [ctypes.c_bool]
    return f


def test_score_ranges_leave_room_on_the_cu(kernels):
    # Where too few (instance, slab) pairs fill the chip, a range must not be so
    # long that its column sums leave a CU one workgroup of four waves for two
    # while workgroups wait, unless no number of ranges that the workspace holds is
    # short enough.
    lds = {k: max(x[".group_segment_fixed_size"] for x in ks)
           for k, ks in _score_kernels(kernels).items()}

    def places(d, n, N):
        keys = (-(-N // n) + 31) // 32 * 32
        need = lds[d, 4, "fused" if n == 1 else "pass2"] + 8 * keys
        return min(2, LDS // (-(-need // LDS_STEP) * LDS_STEP))

    plan = _score_plan()
    rng = random.Random(5)
    sizes = [(250, 4096, 128, 128, 4, 64), (400, 2048, 64, 128, 4, 64), (500, 2048, 64, 128, 2, 100)]
    for _ in range(3000):
        sizes.append((rng.randint(1, 511), rng.randint(1500, 6000), rng.randint(1, 256),
                      rng.choice([64, 128]), rng.randint(1, 8), rng.randint(1, 32)))
    for n, K, B, d, G, w in sizes:
        N = K + B
        p = plan(vase.BF16, n, K, B, d, G, w, False)
        q = plan(vase.BF16, n, K, B, d, G, w, True)
        assert (p.bytes, p.off_col, p.n_chunk2) == (q.bytes, q.off_col, q.n_chunk2)
        for x in (p, q):
            assert 1 <= x.n_chunk1 <= x.n_chunk2 and x.split_keys * x.n_chunk1 >= N
            assert x.split_keys * (x.n_chunk1 - 1) < N and x.split_keys % 32 == 0
        assert p.waves == 4 and p.n_slab == 1
        if places(d, p.n_chunk1, N) == 1 and n * p.n_chunk1 > 256:
            assert all(places(d, m, N) == 1 for m in range(p.n_chunk1, p.n_chunk2 + 1)), (n, K, B, d)


@pytest.mark.parametrize("n,K,B,G,w,ranges", [(233, 4699, 170, 7, 87, 3), (95, 532, 228, 7, 239, 1)])
def test_ranges_of_uneven_slabs(n, K, B, G, w, ranges):
    # full slabs and one that is not: their workgroups do not end together.  Measured at
    # d = 128: 577 us in one range and 544 in three; 119 in two and 98 in one
    assert _score_plan()(vase.BF16, n, K, B, 128, G, w, False).n_chunk1 == ranges
