"""What the built kernels take of a CU, read from the metadata of the library's own
code objects (CPU only)."""
import pytest

from paper_2606_03928_amd import vase


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


def test_no_kernel_spills_registers(kernels):
    assert not {n: k[".vgpr_spill_count"] for n, k in kernels.items() if k[".vgpr_spill_count"]}

