"""What the compiler makes of the search's inner loops (CPU: cross-compiled
to gfx950 assembly and read there).

A row of 16-bit values is read in two 16-byte pieces per lane (65 to 128
values).  If the second piece is loaded only after the first has arrived,
each gather step waits for memory twice, which no result shows: so the
assembly must not wait between the two loads.  And the entry gathers, which
keep two steps in flight, must not wait for a step's rows where they load
them."""
import os
import re
import subprocess

import pytest

from paper_2608_16491_amd import _build

# the entry points of one query, as entry mode 0's kernel evaluates a chunk
PROBE = """
#include "search_common.h"
namespace frog {
template <int C, int LP, typename XT>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(3)))
void entry_probe(DevIndex ix, SearchLaunch a, const int32_t* lr, int lds, uint64_t* out) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    WaveLds<LP> W(smem, lds, 0, ix.dp);
    QueryCtx<C, XT> Q;
    Q.load(ix, a, lr, blockIdx.x);
    Q.load_vector(ix, W.qbuf);
    Pool<LP> pool;
    entry_chunk<C, LP, XT>(ix, a, Q, 0, Q.ne, pool, W);
    for (int s = 0; s < LP; ++s) out[((int64_t)blockIdx.x * LP + s) * 64 + lane_id()] = pool.key[s];
}
template __global__ void entry_probe<4, 1, __half>(DevIndex, SearchLaunch, const int32_t*, int, uint64_t*);
template __global__ void entry_probe<4, 1, bf16x>(DevIndex, SearchLaunch, const int32_t*, int, uint64_t*);
}
"""


def _functions(src):
    """Assembly of each kernel of a HIP source: {demangled name: text}."""
    cmd = [_build.HIPCC, "-O3", "-std=c++17", f"--offload-arch={_build.ARCH}", *_build.DEVICE_FLAGS, "-ffp-contract=off",
           f"-I{_build.INCLUDE}", f"-I{_build.CSRC}", "--cuda-device-only", "-S", "-o", "-", src]
    asm = subprocess.run(cmd, check=True, capture_output=True, text=True).stdout
    found = re.findall(r"^(_ZN\S+):.*?\n(.*?)^\.Lfunc_end", asm, re.S | re.M)
    names = subprocess.run(["c++filt"], input="\n".join(n for n, _ in found), check=True, capture_output=True,
                           text=True).stdout.splitlines()
    short = [re.sub(r"frog::|\(anonymous namespace\)::|void ", "", n).split("(")[0] for n in names]
    return dict(zip(short, (t for _, t in found)))


@pytest.fixture(scope="module")
def traversal():
    return _functions(os.path.join(_build.CSRC, "search_trav.hip"))


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    p = tmp_path_factory.mktemp("probe") / "probe.hip"
    p.write_text(PROBE)
    return _functions(str(p))


def _row_loads(text):
    """Per basic block: L for a 16-byte load, w for a wait on loads."""
    ev = re.findall(r"(global_load_dwordx4|s_waitcnt[^\n]*vmcnt|^\.LBB\S+:)", text, re.M)
    s = "".join("L" if e.startswith("g") else ("|" if e.startswith(".") else "w") for e in ev)
    return [b for b in s.split("|") if "L" in b]


@pytest.mark.parametrize("rows", ["__half", "bf16x"])
@pytest.mark.parametrize("lp", [1, 2, 4])
def test_traversal_loads_rows_whole(traversal, lp, rows):
    blocks = _row_loads(traversal[f"s_search_kernel<4, {lp}, {rows}, true>"])
    assert any("LL" in b for b in blocks)
    for b in blocks:
        # (a wait may stand between two rows, not inside one)
        assert all(len(r) % 2 == 0 for r in re.findall(r"L+", b)), b


@pytest.mark.parametrize("rows", ["__half", "bf16x"])
def test_entry_gather_keeps_two_steps_in_flight(probe, rows):
    blocks = _row_loads(probe[f"entry_probe<4, 1, {rows}>"])
    assert blocks
    for b in blocks:
        assert "LLLL" in b and "Lw" not in b, b


@pytest.mark.parametrize("rows,c", [("float", 2), ("float", 4), ("bf16x", 4)])
@pytest.mark.parametrize("lp", [1, 2, 4])
def test_insertion_branches_once(traversal, lp, rows, c):
    # from the head of the innermost loop that shifts the pool to its last
    # shift: one test, whether the key is there already (lanes masked off by
    # the moves themselves are no tests)
    text = traversal[f"s_search_kernel<{c}, {lp}, {rows}, true>"]
    shifts = [m.start() for m in re.finditer("wave_shr", text)]
    assert len(shifts) >= 2 * lp
    heads = [m.start() for m in re.finditer("Inner Loop Header", text) if m.start() < shifts[0]]
    last = shifts[2 * lp - 1]
    assert text.count("wave_shr", heads[-1], last) == 2 * lp - 1
    assert len(re.findall(r"s_cbranch_(?:scc|vcc)", text[heads[-1]:last])) <= 1
