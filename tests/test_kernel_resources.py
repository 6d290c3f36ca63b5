"""The near-field kernels, bound by vector issue, keep their values in registers:
none has scratch memory (from the metadata of the built library)."""
import os

import pytest

msgpack = pytest.importorskip("msgpack")


def kernels():
    from paper_2512_09478_amd import _lib
    if not os.path.exists(_lib.LIB_PATH):
        from paper_2512_09478_amd import build
        build.build()
    data = open(_lib.LIB_PATH, "rb").read()
    out, at = {}, data.find(b"\xaeamdhsa.kernels")
    while at >= 0:
        u = msgpack.Unpacker(raw=False, strict_map_key=False)
        u.feed(data[at - 1:at + (1 << 20)])   # the map that begins with this key
        for k in u.unpack()["amdhsa.kernels"]:
            out[k[".name"]] = k
        at = data.find(b"\xaeamdhsa.kernels", at + 1)
    return out


def test_near_field_kernels_use_no_scratch():
    near = {n: k for n, k in kernels().items() if "k_p2p" in n}
    assert len(near) == 8   # forward and backward with and without keys, dipoles, gradient twice, Stokes
    for n, k in near.items():
        assert k[".private_segment_fixed_size"] == 0 and k.get(".vgpr_spill_count", 0) == 0, n
