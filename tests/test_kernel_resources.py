"""Registers and scratch of the built kernels, from the metadata the compiler puts beside them.  No GPU."""
import os
import re
import struct
import subprocess

import pytest


@pytest.fixture(scope="module")
def kernels():
    msgpack = pytest.importorskip("msgpack")
    import paper_2512_19342_amd as pkg
    if not os.path.exists(pkg.lib_path()):
        from paper_2512_19342_amd import build
        build.build()
    blob, found, at = open(pkg.lib_path(), "rb").read(), [], 0
    while (at := blob.find(b"AMDGPU\0\0", at)) >= 0:              # a note's name, behind its three sizes
        name, size, kind = struct.unpack_from("<III", blob, at - 12)
        if name == 7 and kind == 32:
            found += msgpack.unpackb(blob[at + 8:at + 8 + size], strict_map_key=False)["amdhsa.kernels"]
        at += 8
    assert found
    names = subprocess.run(["c++filt"], input="\n".join(k[".name"] for k in found), text=True, capture_output=True).stdout.splitlines()
    # "pool_stream<32, 0, ...>" out of "void (anonymous namespace)::pool_stream<32, 0, ...>((anonymous namespace)::DevDesc, ...)"
    short = [re.match(r"(?:void )?([^<(]*(?:<.*?>(?=\())?)", n.replace("(anonymous namespace)::", ""))[1] for n in names]
    assert len(set(short)) == len(short)
    return dict(zip(short, found))


def test_pooling_kernels_spill_only_where_it_was_measured(kernels):
    """A spilled register is reloaded behind a wait for every block of a group's rows; only the 32-lane half-precision kernel
    with three stores is faster that way than with a wavefront less."""
    pools = {n: k for n, k in kernels.items() if n.startswith("pool_")}
    assert len(pools) > 100
    spilling = {n for n, k in pools.items() if k[".private_segment_fixed_size"] or k.get(".vgpr_spill_count")}
    assert all(re.match(r"pool_stream<32, 1, 16, 8, false, false, false, [123]>", n) for n in spilling), spilling   # not the ring


def test_one_launch_steps_do_not_spill(kernels):
    steps = {n: k for n, k in kernels.items() if n.startswith("step_tablewise<")}
    assert len(steps) == 56 and not [n for n, k in steps.items() if k[".private_segment_fixed_size"] or k.get(".vgpr_spill_count")]


def test_three_stores_keep_the_plain_kernels_wavefronts(kernels):
    """fp32 rows of 16 bytes a lane: at most 80 registers, six wavefronts per SIMD."""
    three = [k for n, k in kernels.items() if re.match(r"pool_stream<(8|16|32|64), 0, 16, 8, false, false, ", n)]
    assert len(three) >= 8 and all(k[".vgpr_count"] <= 80 for k in three)


def test_interaction_kernels_do_not_spill(kernels):
    inter = {n: k for n, k in kernels.items() if n.startswith("interact_")}
    assert inter and not [n for n, k in inter.items() if k[".private_segment_fixed_size"] or k.get(".vgpr_spill_count")]
