"""Code sizes of the built kernels.  Two CUs share an instruction cache of 64 KB.  A program of several layers runs a
kernel's code once and then another's, so code that leaves no room for a neighbour is fetched from the L2 again on every
call: with 29 to 35 KB in place of 13 to 21 the fused kernels of a ResNet's layers took 3 to 5 us more, which no
repetition of one layer shows."""
import re
import struct


def kernels(lib):
    """(symbol, bytes of code) of the gfx950 code objects inside the library."""
    data = open(lib, "rb").read()
    for start in (m.start() for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data)):
        count, at = struct.unpack_from("<Q", data, start + 24)[0], start + 32
        for _ in range(count):
            offset, size, name = struct.unpack_from("<QQQ", data, at)
            triple, at = data[at + 24:at + 24 + name], at + 24 + name
            if b"gfx950" in triple and size:
                yield from symbols(data[start + offset:start + offset + size])


def symbols(elf):
    assert elf[:5] == b"\x7fELF\x02"
    shoff, shentsize, shnum = struct.unpack_from("<Q", elf, 40)[0], *struct.unpack_from("<HH", elf, 58)
    sections = [struct.unpack_from("<IIQQQQIIQQ", elf, shoff + i * shentsize) for i in range(shnum)]
    for _, kind, _, _, offset, size, link, _, _, entsize in sections:
        if kind != 2:   # the symbol table
            continue
        names = sections[link][4]
        for at in range(offset, offset + size, entsize):
            name, info, _, _, _, length = struct.unpack_from("<IBBHQQ", elf, at)
            if info & 15 == 2:   # a function
                yield elf[names + name:elf.index(b"\0", names + name)].decode(), length


def test_a_fused_kernel_leaves_half_of_the_instruction_cache_to_its_neighbour(wq):
    sizes = {n: s for n, s in kernels(wq.LIB_PATH) if "k_contract_output" in n}
    # the sixth template argument is DUMP: instances of the debug entry point are nobody's neighbours
    timed = {n: s for n, s in sizes.items() if not re.search(r"k_contract_outputILi\dE(Lb[01]E){4}Lb1E", n)}
    assert len(timed) > 60 and len(timed) < len(sizes)
    large = {n: s for n, s in timed.items() if s > 32768}
    assert not large, large
