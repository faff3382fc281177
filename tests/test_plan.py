"""The launch plans (retopk_plan.h) over whole ranges of sizes, on the CPU: how the
rows of a call are split over blocks.  The header is plain arithmetic; it is compiled
here with g++ and called through ctypes."""
import ctypes as C
import heapq
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2607_27692_amd", "csrc")
SOURCE = """
#include "retopk_plan.h"
using namespace retopk;
extern "C" {
int t_wave_rows(long g, long len, int d) { return dense_wave_rows(g, len, d); }
long t_wave_chunks(long g, long max_len) { return dense_wave_chunks(g, max_len); }
int t_f32_rows(long g, long len) { return dense_f32_rows(g, len); }
long t_f32_chunks(long g, long max_len) { return dense_f32_chunks(g, max_len); }
void t_prefill_plan(long heads, int G, long K, long n, long len, long *out)
{
    const PrefillPlan p = prefill_plan(heads, G, K, n, len);
    const long v[] = {p.cap, p.rows16, p.row_bytes, p.positions, p.lists, p.again_at, p.over_at, p.bytes};
    for (int i = 0; i < 8; ++i) out[i] = v[i];
}
void t_prefill_grid(long cols, long groups, long rows, long *out)
{
    const PrefillGrid g = prefill_grid(cols, groups, rows);
    const long v[] = {g.wc, g.col_blocks, g.chunks, g.chunk_rows};
    for (int i = 0; i < 4; ++i) out[i] = v[i];
}
}
"""
CUS = 256            # compute units, one block each
FILL = 160           # blocks that saturate HBM together
ALL_GROUPS = [*range(1, 301), 400, 511, 512, 513, 768, 1024, 1300, 2048]
LENGTHS = [1, 31, 255, 256, 257, 600, 1024, 2048, 4099, 9000, 16384, 16385, 65536, 131072, 131073,
           242871, 524288, 1 << 20, (1 << 24) - 1, 1 << 24]


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, lib = d / "plan.cpp", d / "plan.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC,
                    str(src), "-o", str(lib)], check=True)
    p = C.CDLL(str(lib))
    for name, args in (("t_wave_rows", (C.c_long, C.c_long, C.c_int)),
                       ("t_wave_chunks", (C.c_long, C.c_long)), ("t_f32_rows", (C.c_long, C.c_long)),
                       ("t_f32_chunks", (C.c_long, C.c_long))):
        fn = getattr(p, name)
        fn.argtypes, fn.restype = args, C.c_long
    out = (C.c_long * 8)()
    p.t_prefill_plan.argtypes = (C.c_long, C.c_int, C.c_long, C.c_long, C.c_long, C.c_void_p)
    p.t_prefill_grid.argtypes = (C.c_long, C.c_long, C.c_long, C.c_void_p)

    def prefill_plan(*args):
        p.t_prefill_plan(*args, out)
        return dict(zip(("cap", "rows16", "row_bytes", "positions", "lists", "again_at", "over_at",
                         "bytes"), out))

    def prefill_grid(*args):
        p.t_prefill_grid(*args, out)
        return dict(zip(("wc", "col_blocks", "chunks", "chunk_rows"), out))

    p.prefill_plan, p.prefill_grid = prefill_plan, prefill_grid
    return p


def makespan(blocks, cus=CUS, fill=FILL):
    """Time of blocks (their rows, in dispatch order) on `cus` slots that share a
    bandwidth of one row per unit, which `fill` of them together can use up."""
    running, t, progress = [], 0.0, 0.0
    todo = iter(blocks)
    nxt = next(todo, None)
    while nxt is not None or running:
        while nxt is not None and len(running) < cus:
            heapq.heappush(running, progress + nxt)
            nxt = next(todo, None)
        end = heapq.heappop(running)
        t += (end - progress) * max(len(running) + 1, fill)
        progress = end
    return t


def chunks(length, rows):
    return [min(rows, length - r) for r in range(0, length, rows)]


# 4096 rows of more than 256 groups: each further round costs a start of some 100 rows,
# so that the split stops at coarser chunks
@pytest.mark.parametrize("length, limit", [(4096, 1.3), (16384, 1.12), (131073, 1.12), (1 << 20, 1.12)])
def test_dense_wave_chunks_are_balanced(plan, length, limit):
    """bf16 full attention of any number of KV groups that gives every slot work of its
    own: the time of its blocks is near that of perfectly divisible work."""
    for groups in ALL_GROUPS:
        if groups * length < FILL * 2048 or groups * length > 1 << 28:
            continue
        for d in (64, 128):
            rows = plan.t_wave_rows(groups, length, d)
            t = makespan(chunks(length, rows) * groups)
            assert t <= limit * groups * length, (
                f"{groups} groups of {length} rows, d={d}: chunks of {rows}, "
                f"{groups * -(-length // rows)} blocks, {t / groups / length:.2f} of the ideal time")


@pytest.mark.parametrize("d", [64, 128])
def test_dense_wave_chunks_do_not_collide(plan, d):
    """Chunks of bf16 rows that start j MiB apart, give or take j * 8 KiB, meet on the
    same memory channels: no length gets such a chunk size."""
    for groups in (1, 2, 4, 6, 8, 12, 24, 40, 130, 264):
        for length in [*range(3000, 1 << 21, 4999), 240 * 4064, 240 * 4128, 30 * 8128, 30 * 8160, 242871]:
            rows = plan.t_wave_rows(groups, length, d)
            stride = rows * 2 * d
            j = (stride + (1 << 19)) >> 20
            assert j == 0 or abs(stride - (j << 20)) > j * 8192, f"{groups} groups of {length}: chunks of {rows}"


def test_dense_f32_chunks_split_only_to_fill(plan):
    """f32 full attention takes chunks of fewer than 1024 rows only where they still
    leave at most one block per CU."""
    for groups in ALL_GROUPS:
        for length in LENGTHS:
            rows = plan.t_f32_rows(groups, length)
            assert rows == 1024 or groups * -(-length // rows) <= CUS, (groups, length, rows)
            assert rows == 256 or groups * -(-length // (rows // 2)) > CUS, (groups, length, rows)


@pytest.mark.parametrize("kind", ["wave", "f32"])
def test_dense_chunk_limits(plan, kind):
    """Chunks stay inside the kernels' limits, and no length up to max_len has more of
    them than the workspace holds."""
    for groups in ALL_GROUPS:
        for i, max_len in enumerate(LENGTHS):
            room = (plan.t_wave_chunks if kind == "wave" else plan.t_f32_chunks)(groups, max_len)
            for length in LENGTHS[:i + 1]:
                if kind == "wave":
                    for d in (64, 128):
                        rows = plan.t_wave_rows(groups, length, d)
                        assert rows % 32 == 0 and 256 <= rows <= 1 << 17
                        assert -(-length // rows) <= room, (groups, length, max_len)
                else:
                    rows = plan.t_f32_rows(groups, length)
                    assert rows in (256, 512, 1024)
                    assert -(-length // rows) <= room, (groups, length, max_len)


START_ROWS = 170     # what the start of a k_pf_scan block costs, in rows


# at 16K rows, chunks for another round would be shorter than their start is worth
@pytest.mark.parametrize("rows, limit", [(16384, 1.25), (65536, 1.12), (131072, 1.12), (131600, 1.12),
                                         (1 << 20, 1.12)])
def test_prefill_grid_is_balanced(plan, rows, limit):
    """k_pf_scan for any number of KV groups and virtual queries: the time of its blocks,
    placed on the 8 XCDs in turn, is near that of evenly divided work."""
    for groups in [*range(1, 41), 56, 72, 96, 130, 200, 256, 257, 264, 400, 2048]:
        for cols in (1, 16, 128, 130, 256, 640, 1024, 1025, 1792, 3072, 4096, 32768):
            g = plan.prefill_grid(cols, groups, rows)
            work = groups * g["col_blocks"] * rows
            if work < CUS * 2048 or work > 1 << 25:
                continue
            pairs = groups * g["chunks"]
            sizes = chunks(rows, g["chunk_rows"])
            assert len(sizes) == g["chunks"] and g["wc"] * g["col_blocks"] * 128 >= cols
            worst = 0.0
            for xcd in range(8):
                blocks = [sizes[pair % g["chunks"]] + START_ROWS for pair in range(xcd, pairs, 8)
                          for _ in range(g["col_blocks"])]
                worst = max(worst, makespan(blocks, CUS // 8, CUS // 8) * 8)
            assert worst <= limit * (work + CUS * START_ROWS), (
                f"{groups} groups, {cols} queries, {rows} rows: {g}, {worst / work:.2f} of the ideal time")


def test_prefill_plan_limits(plan):
    """Workspaces are bounded, and a launch's lists or score rows fit them."""
    for heads, G in ((1, 1), (4, 4), (28, 7), (32, 4), (40, 5), (64, 1), (2048, 8)):
        for K in (1, 64, 512, 513, 2048):
            for n in (2, 32, 512, 4096):
                for length in (n, 4095, 4096, 8175, 8176, 8192, 16384, 32768, 131072, 1 << 24):
                    if length < n:
                        continue
                    p = plan.prefill_plan(heads, G, K, n, length)
                    assert 1 <= p["positions"] <= n
                    assert p["again_at"] >= heads * (p["row_bytes"] + 8) * p["positions"]
                    assert p["again_at"] % 8 == 0 and p["over_at"] % 4 == 0
                    assert p["over_at"] >= p["again_at"] + 8 * n * heads and p["bytes"] >= p["over_at"] + 4 * n
                    assert p["again_at"] <= max(257 << 20, heads * (p["row_bytes"] + 8) + 256)
                    if p["lists"]:
                        assert p["row_bytes"] == 8 * p["cap"] and p["cap"] >= 8 * K
                    else:
                        assert p["row_bytes"] >= 4 * p["rows16"]
