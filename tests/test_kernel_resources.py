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


def test_kernel_of_narrow_slices_has_hardly_any_shared_memory_beside_what_its_launch_asks_for():
    """The dispatch takes k_small_cols for several tokens where its launch asks for at most half of a compute unit's 160 KB, so that
    two workgroups share one: a fixed part beside it would leave layers just below the line with one. With the router's logits
    (mode 0) the choices of eight wavefronts, 512 bytes."""
    fixed = {n: k[".group_segment_fixed_size"] for n, k in kernels().items() if "k_small_cols" in n}
    assert len(fixed) == 12
    for name, size in fixed.items():
        mode = int(re.search(r"k_small_colsILb[01]ELi(\d)E", name).group(1))
        assert size <= (512 if mode == 0 else 0), (name, size)
