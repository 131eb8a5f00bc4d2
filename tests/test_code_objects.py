"""What the compiler made of the kernels, from the metadata in the built library."""
import pytest

from paper_2405_01481_amd import rollout as R

msgpack = pytest.importorskip("msgpack")


def _kernels():
    """Metadata of every kernel: the value of the key amdhsa.kernels of each code object's note."""
    R.lib()
    with open(R.LIB_PATH, "rb") as f:
        data = f.read()
    key, i = b"\xaeamdhsa.kernels", 0
    while (i := data.find(key, i)) >= 0:
        u = msgpack.Unpacker(raw=False, strict_map_key=False, max_buffer_size=1 << 28)
        u.feed(data[i - 1:i + (1 << 24)])          # the map's header is one byte
        yield from u.unpack()["amdhsa.kernels"]
        i += len(key)


def test_decode_attention_uses_no_scratch():
    """Its loop keeps two pages, the output and the queries in registers; what does not fit is written to memory and read back
    on every page."""
    found = {k[".name"]: (k[".private_segment_fixed_size"], k[".vgpr_spill_count"]) for k in _kernels() if "attn_decode_kernel" in k[".name"]}
    assert len(found) >= 12                        # two head dimensions, two wave counts, plain, consumer and pair form
    assert {n: v for n, v in found.items() if v != (0, 0)} == {}
