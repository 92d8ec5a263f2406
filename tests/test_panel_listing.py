"""What the compiler made of the panel kernel's written-out products (no GPU).  It does not know how long such a product takes,
so it has to leave alone what the kernel's order rests on: nothing of a wave in memory, no tile moved about in the loop, idle
states between whatever touches a tile and the products, on the way in and on the way out."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2511_20340_amd import binding as sfb

LLVM = "/opt/rocm/llvm/bin"
TILES = {(10, 8, 2), (8, 8, 2), (6, 8, 2), (4, 8, 3), (4, 4, 4), (5, 4, 2), (5, 4, 4)}   # a wave's tiles, slices in LDS


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{(TM, TN, STAGES): (code lines, notes of its code object)} of the built library's panel kernels."""
    d = tmp_path_factory.mktemp("listing")
    shutil.copy(sfb.LIB_PATH, d / "lib.so")
    run = lambda *a: subprocess.run(a, cwd=d, capture_output=True, text=True, check=True).stdout
    run(f"{LLVM}/llvm-objdump", "--offloading", "lib.so")
    found = {}
    for f in sorted(os.listdir(d)):
        if "gfx950" not in f or b"gemm_panel_kernel" not in (d / f).read_bytes():
            continue
        notes = run(f"{LLVM}/llvm-readelf", "--notes", f)
        for name, body in re.findall(r"^[0-9a-f]+ <(\S*gemm_panel_kernel\S*)>:\n(.*?)(?=^[0-9a-f]+ <|\Z)",
                                     run(f"{LLVM}/llvm-objdump", "-d", f), re.M | re.S):
            tile = tuple(map(int, re.findall(r"Li(\d+)E", name)))[2:]
            code = [m.groups() for m in re.finditer(r"^\t(\S.*?)\s*// ([0-9A-F]{12}):", body, re.M)]
            meta = notes[:notes.index(f".symbol:         {name}.kd")].rsplit("- .agpr_count", 1)[1]
            rest = notes[notes.index(f".symbol:         {name}.kd"):].split("- .agpr_count", 1)[0]
            found[tile] = ([(c, int(a, 16)) for c, a in code], meta + rest)
    assert set(found) == TILES
    return found


def registers(operand):
    m = re.fullmatch(r"([va])\[(\d+):(\d+)\]|([va])(\d+)", operand)
    if not m:
        return set()
    if m[1]:
        return {(m[1], i) for i in range(int(m[2]), int(m[3]) + 1)}
    return {(m[4], int(m[5]))}


def operands(line):
    return [o.strip() for o in line.split(" ", 1)[1].split(",")] if " " in line else []


def touched(line):
    return set().union(*(registers(o.split(" ")[0]) for o in operands(line)), set())


@pytest.mark.parametrize("tile", sorted(TILES))
def test_products_are_left_alone(kernels, tile):
    code, notes = kernels[tile]
    for field in ("private_segment_fixed_size", "vgpr_spill_count"):
        assert re.findall(rf"\.{field}:\s*(\d+)", notes) == ["0"], field
    first = next(i for i, (c, _) in enumerate(code) if c.startswith("v_mfma"))
    last = max(i for i, (c, _) in enumerate(code) if c.startswith("v_mfma"))
    products = [c for c, _ in code[first:last + 1] if c.startswith("v_mfma")]
    assert len(products) == 2 * tile[0] * tile[1]                      # the loop's two k-steps, once
    tiles = set().union(*(registers(operands(c)[0]) for c in products))
    inputs = set().union(*(registers(o) for c in products for o in operands(c)[1:3]))
    assert len(tiles) == 4 * tile[0] * tile[1] and not tiles & inputs  # every tile in place, from product to product
    assert all(registers(operands(c)[0]) == registers(operands(c)[3]) for c in products)

    # the loop, its branch included, twice round: no other vector instruction reads or writes a tile, and what one writes to a
    # register is not a product's input (such registers hold addresses between one fragment and the next)
    end = next(i for i in range(last, len(code)) if code[i][0].startswith("s_cbranch"))
    written = set()
    for c, _ in 2 * code[first:end + 1]:
        if c.startswith("v_mfma"):
            assert not written & inputs & set().union(*(registers(o) for o in operands(c)[1:3])), c
        elif c.startswith("ds_read"):
            assert not touched(c) & tiles, c
            written -= registers(operands(c)[0])
        elif not c.startswith(("s_", "buffer_load")):
            assert c.startswith("v_") and not touched(c) & tiles, c
            written |= registers(operands(c)[0])

    # on the way out: nothing touches a tile before the idle states
    idle = next(i for i in range(last, len(code)) if code[i][0] == "s_nop 15")
    assert [c for c, _ in code[idle:idle + 2]] == ["s_nop 15"] * 2
    assert not any(touched(c) & tiles for c, _ in code[last + 1:idle])
    # on the way in: nothing touches a tile behind them
    idle = max(i for i in range(first) if code[i][0] == "s_nop 7")
    assert not any(touched(c) & tiles for c, _ in code[idle:first])
