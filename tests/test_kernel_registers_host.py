"""The scan's kernels keep their values in registers: a reload from scratch memory would wait for every key tile in flight. Read from the
metadata of the built library's code objects."""
import msgpack

from paper_2602_08686_amd import build

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _kernels():
    """name -> metadata of every gfx950 kernel in the library."""
    blob, out, at = build.LIB.read_bytes(), {}, 0
    number = lambda p: int.from_bytes(blob[p:p + 8], "little")  # noqa: E731
    while (at := blob.find(MAGIC, at)) >= 0:
        p = at + len(MAGIC) + 8
        for _ in range(number(p - 8)):
            offset, size, length = number(p), number(p + 8), number(p + 16)
            target, p = blob[p + 24:p + 24 + length], p + 24 + length
            if not target.endswith(b"gfx950"):
                continue
            elf = blob[at + offset:at + offset + size]
            note = elf.find(b"AMDGPU\0")   # the note: length of its name, of its contents, type 32, name, contents
            contents = int.from_bytes(elf[note - 8:note - 4], "little")
            assert note > 0 and elf[note - 4:note] == (32).to_bytes(4, "little")
            meta = msgpack.unpackb(elf[note + 8:note + 8 + contents])
            out.update({k[".name"]: k for k in meta["amdhsa.kernels"]})
        at += len(MAGIC)
    return out


def test_no_scan_kernel_has_scratch_memory():
    kernels = _kernels()
    scan = {n: k for n, k in kernels.items() if any(f in n for f in ("scan_short_kernel", "rowstats_lds_kernel", "colsum_lds_kernel"))}
    assert len(scan) > 60 and sum("scan_short_kernel" in n for n in scan) > 20, len(scan)
    spilled = {n: k[".private_segment_fixed_size"] for n, k in scan.items() if k[".private_segment_fixed_size"]}
    assert not spilled, spilled
