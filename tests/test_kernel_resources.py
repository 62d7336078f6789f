"""What the compiler gave the kernels of the built library (its own metadata, read on the host): registers that spill and fixed
shared memory, where the code counts on them."""
import re

import pytest

from paper_2308_14352_amd import binding as B

msgpack = pytest.importorskip("msgpack")


def kernels():
    """{mangled name: metadata} of every kernel in the library."""
    B.lib()                                          # (builds it if there is none)
    data, out = open(B.LIB_PATH, "rb").read(), {}
    for m in re.finditer(re.escape(b"\xaeamdhsa.kernels"), data):
        unpacker = msgpack.Unpacker(raw=False, strict_map_key=False)
        unpacker.feed(data[m.start() - 1:m.start() + (4 << 20)])
        out.update((k[".name"], k) for k in unpacker.unpack()["amdhsa.kernels"])
    return out


def test_streaming_decode_kernel_keeps_its_loop_in_registers():
    """Two sets of loads, the digits of x for all three bitwidths and the records of the chosen experts live through the loop of
    k_moe_stream: a register of the sets or digits that spills is loaded again for every block (4 to 6 % of a call with eleven)."""
    spilled = {n: k[".vgpr_spill_count"] for n, k in kernels().items() if "k_moe_stream" in n}
    assert len(spilled) == 10 and max(spilled.values()) <= 1, spilled
