"""Properties of the device code that no result shows, checked on its
assembly (CPU only): small kernels that call one helper each are compiled for
gfx950 and their memory instructions read."""

import os
import re
import subprocess

import pytest

from paper_1412_7789_amd import build as lib_build

HIPCC = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")


def instructions(tmp_path, source, also="buffer_"):
    """The memory instructions of the kernels in `source`, which may use
    filtered.hpp, and those that start with `also`."""
    src, asm = tmp_path / "snippet.hip", tmp_path / "snippet.s"
    src.write_text('#include "filtered.hpp"\nusing namespace pfac;\nusing namespace pfac::dev;\n' + source)
    subprocess.run([HIPCC, *lib_build.HIPCC_FLAGS, f"-I{lib_build.INCLUDE}", f"-I{lib_build.CSRC}", "-x", "hip",
                    "--cuda-device-only", "-S", str(src), "-o", str(asm)], check=True, capture_output=True, text=True)
    lines = (line.split(";")[0].strip() for line in asm.read_text().splitlines())
    return [line for line in lines if re.match(r"(buffer|global|flat)_|" + also, line)]


@pytest.mark.parametrize("segs", [1, 2, 4])
def test_text_loads_carry_their_offset_where_it_is_checked(tmp_path, segs):
    """A chunk's descriptor ends with the text, and a raw buffer load is checked
    against it by the vector offset plus the immediate, never by the scalar
    offset, which must be 0: in the whole-chunk loads and in the slow mode's
    loads of one segment, for a segment index known only at run time."""
    loads = [i for i in instructions(tmp_path, f"""
__global__ void whole(FilterLaunch F, int64_t c, uint32_t *out) {{
    ChunkRegs<{segs}> R;
    load_chunk<{segs}>(F, c, lane_id(), R);
    uint32_t x = R.tail;
    for (int j = 0; j < {segs}; ++j) x ^= R.d[j][0] ^ R.d[j][1] ^ R.d[j][2] ^ R.d[j][3];
    out[threadIdx.x] = x;
}}
__global__ void one(FilterLaunch F, int64_t c, int j, uint32_t *out) {{
    ChunkRegs<1> R;
    load_segment<{segs}>(F, c, j, lane_id(), R);
    out[threadIdx.x] = R.tail ^ R.d[0][0] ^ R.d[0][1] ^ R.d[0][2] ^ R.d[0][3];
}}
""") if i.startswith("buffer_load")]
    assert len(loads) == segs + 1 + 2
    for i in loads:
        # buffer_load_x vdata, vaddr | off, s[descriptor], soffset [offen] [offset:n] [nt]
        m = re.match(r"buffer_load_\w+ \S+, (\S+), s\[\d+:\d+\], (\S+)(.*)", i)
        assert m, i
        assert m.group(2) == "0", i
        assert m.group(1) == "off" or "offen" in m.group(3), i


def test_matches_for_the_host_are_released_before_the_count(tmp_path):
    """The host reads a dispatched call's pinned match arrays as soon as the
    count is reported, before the kernel's end: every block releases its matches
    to the system (a cache writeback at system scope) before it counts itself
    done, only where there are such arrays."""
    code = instructions(tmp_path, """
__global__ void report(ScanArgs S) { report_count(S); }
""", also="s_cbranch")
    release = code.index("buffer_wbl2 sc0 sc1")
    done = next(i for i, line in enumerate(code) if "atomic_add" in line)
    assert release < done
    assert code[release - 1].startswith("s_cbranch"), "a scan without pinned arrays needs no writeback"
