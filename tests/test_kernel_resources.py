"""Registers that the compiler reports for the library's kernels (the metadata notes of libgspc.so's own code objects)."""
import ctypes
import struct

import pytest

from paper_2006_09791_amd import binding as b

msgpack = pytest.importorskip("msgpack")


def kernels():
    """Mangled name -> metadata of every kernel in the library."""
    data, found, at = open(b.LIB_PATH, "rb").read(), {}, 0
    while (at := data.find(b"\x7fELF\x02\x01\x01\x40", at)) >= 0:      # an embedded code object
        elf = data[at:]
        shoff, = struct.unpack_from("<Q", elf, 40)
        size, count = struct.unpack_from("<HH", elf, 58)
        for i in range(count):
            kind, = struct.unpack_from("<I", elf, shoff + i * size + 4)
            off, left = struct.unpack_from("<QQ", elf, shoff + i * size + 24)
            while kind == 7 and left > 0:                              # notes
                nl, dl, note = struct.unpack_from("<III", elf, off)
                body = off + 12 + (nl + 3) // 4 * 4
                if note == 32:
                    for k in msgpack.unpackb(elf[body:body + dl])["amdhsa.kernels"]:
                        found[k[".name"]] = k
                step = body + (dl + 3) // 4 * 4 - off
                off, left = off + step, left - step
        at += 4
    return found


@pytest.mark.parametrize("form,most", [("Lb0ELb0ELb0E", 24), ("Lb1ELb0ELb0E", 20), ("Lb1ELb1ELb0E", 20)])
def test_large_split_block_keeps_its_scalars(form, most):
    """The block of the large fp32 3x3 layers: kernel arguments that it does not read, put between those that it reads,
    shift its scalar loads and cost it registers (29 spills instead of 18 with even rows and 16-byte stores)."""
    name = "_ZN4gspc11conv_split3ILi2ELi4ELi2ELi2ELi1ELi4ELi1Ef" + form
    k, = [v for n, v in kernels().items() if n.startswith(name)]
    assert k[".sgpr_spill_count"] <= most, k[".sgpr_spill_count"]


def test_split_kernels_need_no_scratch():
    for n, k in kernels().items():
        if "conv_split3" in n or "conv_direct_rows" in n:
            assert k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0, n


@pytest.mark.parametrize("inst", range(5))
def test_split_kernel_refuses_a_plan_without_an_instance(inst):
    """Blocks of more than one filter tile have no instance that splits the filters itself: such a plan is an error and does
    not run on the filter layout of another shape (checked before anything is launched)."""
    launch = b.load()["_ZN4gspc13launch_split3ERKNS_10ConvParamsERKNS_10Split3PlanEP12ihipStream_tPPKc"]
    params, plan, name = (ctypes.c_char * 1024)(), (ctypes.c_int * 256)(), ctypes.c_char_p()
    plan[0], plan[1], plan[2] = inst, 4, 1                              # shape, 32 channels per chunk, unsplit filters
    not_supported = 801                                                # hipErrorNotSupported
    assert launch(params, plan, None, ctypes.byref(name)) == not_supported and not name.value


def waves(k):
    """Waves per SIMD that a kernel's registers leave room for."""
    return min(8, 512 // max(8, (k[".vgpr_count"] + 7) // 8 * 8))


def test_resident_filters_keep_three_blocks_per_compute_unit():
    """Eight tiles per wave, one channel block per chunk at stride 1: LDS leaves room for three blocks and four, and
    a launch that fits by LDS is taken for one round: the registers must leave room for three."""
    k, = [v for n, v in kernels().items() if n.startswith("_ZN4gspc12conv_mfma16wILi2ELi4ELi1ELi1ELb0ELi4E")]
    assert waves(k) >= 3, k[".vgpr_count"]


@pytest.mark.parametrize("shape,least", [("1ELi4ELi1ELi4", 5), ("2ELi4ELi1ELi4", 4), ("2ELi4ELi2ELi2", 4)])
@pytest.mark.parametrize("stride", [1, 2])
def test_bf16_split_blocks_keep_their_waves(shape, least, stride):
    """16 channels per chunk, even rows, 4-byte stores: left to the compiler these are one register past a step."""
    k, = [v for n, v in kernels().items() if n.startswith(f"_ZN4gspc11conv_split3ILi{shape}ELi1ELi2ELi{stride}EtLb1ELb0E")]
    assert waves(k) >= least, k[".vgpr_count"]


def test_bf16_strips_keep_their_waves():
    """bf16 depthwise at stride 2: left to the compiler it is two registers past the step of six waves."""
    k, = [v for n, v in kernels().items() if n.startswith("_ZN4gspc17conv_direct_smallILi1ELi1ELi2ELi2Et")]
    assert waves(k) >= 6 and k[".vgpr_spill_count"] == 0, k[".vgpr_count"]
