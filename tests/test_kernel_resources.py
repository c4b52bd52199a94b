"""What the built kernels take of a CU, read from the metadata of the library's own
code objects (CPU only)."""
import re

import pytest

from paper_2606_03928_amd import vase

KIND = {0: "pass1", 1: "pass2", 2: "fused"}


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

