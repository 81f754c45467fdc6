"""What the compiler makes of loops whose rate depends on it (CPU only: hipcc writes gfx950 assembly without a GPU).

A streaming loop runs at memory speed only while its loads stay in flight.  Changes of the source that look harmless
(a second way to load, a condition around the loads) have made the compiler wait for all of them at once, which no test of
the results shows."""
import functools
import os
import re
import shutil
import subprocess
import tempfile

import pytest

from paper_1511_04561_amd import build

pytestmark = pytest.mark.skipif(not (os.path.exists(build.hipcc()) or shutil.which(build.hipcc())), reason="needs hipcc")

#: kernels of the headers, as explicit instantiations
KERNELS = """
template __global__ void k_absmax_whole<16, 1>(const float *, size_t, size_t, size_t, size_t, size_t, float *);
template __global__ void k_encode<1, 2, 1, false, true, true>(const uint32_t *, const float *, size_t, size_t, size_t, size_t, size_t, size_t, uint32_t, float *, uint8_t *);
template __global__ void k_encode<1, 4, 1, false, true, false>(const uint32_t *, const float *, size_t, size_t, size_t, size_t, size_t, size_t, uint32_t, float *, uint8_t *);
template __global__ void k_encode<4, 4, 1, true, true, false>(const uint32_t *, const float *, size_t, size_t, size_t, size_t, size_t, size_t, uint32_t, float *, uint8_t *);
template __global__ void k_decode_flat<16, 8, 2, 4>(const uint32_t *, const uint8_t *, const float *, uint64_t, uint32_t, uint32_t, uint64_t, uint64_t, uint32_t, uint64_t, uint32_t, float *);
template __global__ void k_seg_encode<false, 8>(const uint32_t *, const float *, size_t, const uint64_t *, uint32_t, size_t, size_t, const float *, uint8_t *);
template __global__ void k_seg_encode<true, 16>(const uint32_t *, const float *, size_t, const uint64_t *, uint32_t, size_t, size_t, const float *, uint8_t *);
template __global__ void k_seg_encode_copied<false, 8>(const uint32_t *, const float *, size_t, const uint64_t *, uint32_t, size_t, size_t, const float *, uint8_t *);
template __global__ void k_seg_encode_copied<true, 16>(const uint32_t *, const float *, size_t, const uint64_t *, uint32_t, size_t, size_t, const float *, uint8_t *);
template __global__ void k_seg_encode_parts<false, 8>(const uint32_t *, const float *, size_t, const uint64_t *, uint32_t, size_t, size_t, const float *, uint32_t, float *, uint8_t *);
template __global__ void k_seg_encode_parts<true, 16>(const uint32_t *, const float *, size_t, const uint64_t *, uint32_t, size_t, size_t, const float *, uint32_t, float *, uint8_t *);
template __global__ void k_error_stats_one<12, true>(const uint32_t *, const float *, size_t, size_t, size_t, float *, const float *, uint32_t, double *);
template __global__ void k_avg_team<8, 1, true, 3, false, false, 4>(const uint32_t *, WorkerPtrs, int, const float *, size_t, size_t, size_t, size_t, size_t, uint32_t, uint32_t, float *, uint8_t *);
void *long_expansion = (void *)k_seg_decode_long;
"""


@functools.lru_cache(maxsize=None)
def assembly():
    """Kernel name without its namespace -> list of basic blocks, each a list of instructions; and -> vector registers."""
    with tempfile.TemporaryDirectory() as d:
        src, out = os.path.join(d, "kernels.hip"), os.path.join(d, "kernels.s")
        with open(src, "w") as f:
            f.write('#include <hip/hip_runtime.h>\n#include "dq8_device.hpp"\n#include "dq8_kernels_codec.hpp"\n#include "dq8_kernels_segments.hpp"\n#include "dq8_kernels_stats.hpp"\n#include "dq8_kernels_avg_encode.hpp"\nnamespace {\n%s}\n' % KERNELS)
        flags = [f for f in build.FLAGS if f != "-shared"]
        subprocess.check_call([build.hipcc()] + flags + ["-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, "-S",
                                                        "--cuda-device-only", "-o", out, src])
        with open(out) as f:
            lines = f.read().split("\n")
    kernels, registers, blocks, name = {}, {}, None, None
    for line in lines:
        m = re.match(r"^(_Z\w+):", line)
        if m:
            name = re.sub(r"^_ZN12_GLOBAL__N_1\d\d?", "", m.group(1))
            blocks = kernels.setdefault(name, [[]])
        elif line.startswith("; NumVgprs:"):
            registers[name] = int(line.split(":")[1])
        elif line.startswith(".Lfunc_end"):
            blocks = None
        elif blocks is not None and re.match(r"^\.LBB\w+:", line):
            blocks.append([])
        elif blocks is not None and re.match(r"^\s+(v_|s_|ds_|global_|buffer_|flat_|scratch_)", line):
            blocks[-1].append(line.split(";")[0].strip())
            if blocks[-1][-1].startswith("s_cbranch"):
                blocks.append([])
    return kernels, registers


def kernel(prefix, what=0):
    """Basic blocks (0) or vector registers (1) of a kernel."""
    found = [b for name, b in assembly()[what].items() if name.startswith(prefix)]
    assert len(found) == 1, prefix
    return found[0]


def waits(block):
    """The vmcnt of the block's waits, in order."""
    return [int(m.group(1)) for i in block for m in re.finditer(r"vmcnt\((\d+)\)", i)]


def test_block_maxima_keep_their_loads_in_flight():
    """k_absmax_whole takes its sixteen quads in groups of four and requests each again at once: a wait leaves twelve loads."""
    loops = [b for b in kernel("k_absmax_wholeILi16ELi1E") if sum(i.startswith("global_load_dwordx4") for i in b) == 16 and waits(b)]
    assert sum(min(waits(b)) >= 12 for b in loops) == 1, [waits(b) for b in loops]


def test_compression_requests_the_next_block_before_it_waits():
    """k_encode without conditions around its loads: in its loop a block is requested while the one before it is on its way."""
    slots = []
    for b in kernel("k_encodeILi1ELi2ELi1ELb0ELb1ELb1E")[1:]:
        loads = [i for i, ins in enumerate(b) if ins.startswith("global_load_dwordx4")]
        if len(loads) == 2 and waits(b):  # in the loop, where a block's loads are followed by the wait for the one before
            slots.append(waits(b[:loads[-1]]))
    assert len(slots) == 2 and [] in slots, slots


def test_compression_has_its_table_before_its_loop():
    """k_encode with a wavefront per unit: no load of the search table is left, in any thread, when the workgroup meets in front of the
    loop, whose waits would count it."""
    meet = [b for b in kernel("k_encodeILi1ELi4ELi1ELb0ELb1ELb0E") if any(i.startswith("s_barrier") for i in b)]
    assert len(meet) == 1
    assert any(i.startswith("ds_write_b128") for i in meet[0]) and waits(meet[0])[-1] == 0, meet[0]


def test_teams_have_their_table_before_their_first_unit():
    """k_encode with a team per unit: no unit's loads set out before the workgroup has met over the table."""
    blocks = kernel("k_encodeILi4ELi4ELi1ELb1ELb1ELb0E")
    meet = min(i for i, b in enumerate(blocks) if any(w.startswith("s_barrier") for w in b))
    upto = [w for b in blocks[:meet] for w in b] + blocks[meet][:[w.startswith("s_barrier") for w in blocks[meet]].index(True)]
    loads = [w for w in upto if w.startswith("global_load_dwordx4")]
    assert loads and not any(w.endswith(" nt") for w in loads), loads


def test_expansion_by_position_keeps_no_store_offsets():
    """k_decode_flat: registers of sixteen code words, the scales and a quad, not of sixteen store offsets besides."""
    assert kernel("k_decode_flatILi16ELi8E", 1) <= 76


@pytest.mark.parametrize("marks,waves", [(0, 8), (1, 16)])
def test_segment_compression_leaves_room_for_wavefronts(marks, waves):
    """k_seg_encode: seven wavefronts of it fit the registers of a SIMD, and its code is not several times its loop."""
    name = "k_seg_encodeILb%dELi%dE" % (marks, waves)
    assert kernel(name, 1) <= 72
    assert sum(len(b) for b in kernel(name)) < 3000


@pytest.mark.parametrize("marks,waves", [(0, 8), (1, 16)])
@pytest.mark.parametrize("scales", ["copied", "parts"])
def test_segment_compression_of_usual_sets_leaves_room_for_wavefronts(scales, marks, waves):
    """The same of the forms for up to 1024 segments, whose scales are copied to LDS or formed from parts."""
    name = "k_seg_encode_%sILb%dELi%dE" % (scales, marks, waves)
    assert kernel(name, 1) <= 72
    assert sum(len(b) for b in kernel(name)) < 3000


def loads_of(block, words):
    return sum(i.startswith("global_load_dword%s " % words) for i in block)


def test_statistics_of_one_block_keep_half_a_unit_in_flight():
    """k_error_stats_one: six wavefronts per SIMD, and in its loop a wait for two quads leaves the unit's two others on their way."""
    assert kernel("k_error_stats_oneILi12ELb1E", 1) <= 80
    blocks = kernel("k_error_stats_oneILi12ELb1E")
    last = max(i for i, b in enumerate(blocks) if loads_of(b, "x4") == 2)  # where a half is requested again at the loop's end
    first = min(i for i, b in enumerate(blocks) if waits(b) and loads_of(b, "x4") == 2)  # the other half, in its middle
    assert first < last and loads_of(blocks[first], "x4") == 2
    assert [w for b in blocks[first:last] for w in waits(b)] and min(w for b in blocks[first:last] for w in waits(b)) >= 2


def test_long_sets_are_expanded_a_unit_ahead():
    """k_seg_decode_long: the sixteen words of the next unit are requested together, and sixteen stores follow without a wait."""
    blocks = kernel("k_seg_decode_longE")
    assert sum(loads_of(b, "") == 16 and not waits(b) for b in blocks) >= 3  # before the loop, and for either kind of unit
    assert sum(sum(i.startswith("global_store_dwordx4") for i in b) == 16 and not waits(b) for b in blocks) == 1


def test_averages_compressed_again_request_all_workers_ahead():
    """k_avg_team, eight workers of four words each: in the loop over whole units all are requested again before the first of those that
    are waited for, at any other unit (short ones, any alignment) together."""
    blocks = kernel("k_avg_teamILi8ELi1ELb1ELi3ELb0ELb0ELi4E")
    steady = [b for b in blocks if loads_of(b, "") >= 32 and waits(b)]
    assert len(steady) == 2 and all(max(waits(b)) >= 36 for b in steady), [waits(b) for b in steady]
    assert sum(loads_of(b, "") == 32 and not waits(b) for b in blocks) >= 3  # before the loops, and the two halves of the general one
