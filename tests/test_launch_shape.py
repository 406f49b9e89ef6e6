"""The launch rules (csrc/launch.h), asked through a small driver, and what the compiler made of the kernels they
launch, read from the built library's metadata.  No GPU."""
import os
import re
import shutil
import struct
import subprocess
from collections import namedtuple

import numpy as np
import pytest

import paper_1912_09268_amd as M

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1912_09268_amd", "csrc")
READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"
KINDS = ["pack", "reduce", "update", "reduce_update", "pipeline", "direct"]
DTYPES = ["f32", "bf16", "f16"]
CU_LDS, LDS_GRAIN = 160 << 10, 1280
Kernel = namedtuple("Kernel", "few kind half P form lds vgprs sgprs dtype")
Shape = namedtuple("Shape", "tiles_per_wg units grid xcd_contiguous run_log2 may_be_few form wgs_per_cu rolling in_pieces")


def build_driver(folder, *defines):
    exe = str(folder / "driver")
    r = subprocess.run(["g++", "-std=c++17", "-Wall", "-Wno-unused-function", *(f"-D{d}" for d in defines), "-I", os.path.join(ROOT, "include"),
                        "-I", CSRC, os.path.join(ROOT, "tests", "launch_shape_driver.cpp"), os.path.join(CSRC, "layout.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def ask(lines):
        r = subprocess.run([exe], input="\n".join(lines), capture_output=True, text=True, timeout=60)
        assert r.returncode == 0
        out = [tuple(int(x) for x in line.split()) for line in r.stdout.splitlines()]
        assert len(out) == len(lines)
        return out
    return ask


Form = namedtuple("Form", "form on_lines through may_be_few run_log2")


def forms_of(ask, n_elems, merged, P, dtype, reduced=0):
    """What the rules make of launches over all of a model: a Form for each kind."""
    out = ask([f"forms {P} {DTYPES.index(dtype)} {reduced} {len(n_elems)} " + " ".join(f"{n} {m}" for n, m in zip(n_elems, merged))])[0]
    return {kind: Form(*out[5 * k:5 * k + 5]) for k, kind in enumerate(KINDS)}


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    return build_driver(tmp_path_factory.mktemp("launch"))


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Every kernel of the built library: the code objects in it are bundles of (offset, size, target)."""
    data, found, at = open(M.library_path(), "rb").read(), [], 0
    part = str(tmp_path_factory.mktemp("kernels") / "code")
    while (at := data.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        (n,), pos = struct.unpack_from("<Q", data, at + 24), at + 32
        for _ in range(n):
            offset, size, length = struct.unpack_from("<QQQ", data, pos)
            target = data[pos + 24:pos + 24 + length]
            pos += 24 + length
            if b"gfx950" not in target or size == 0:
                continue
            with open(part, "wb") as f:
                f.write(data[at + offset:at + offset + size])
            notes = subprocess.run([READELF, "--notes", part], capture_output=True, text=True, check=True).stdout
            for text in notes.split("\n  - .a")[1:]:
                m = re.search(r"\.name:\s+\S*mgwfbp_(few|stream)_kernelILi(\d)E(\w+?)Li(\d+)ELi(n?\d)E", text)
                field = lambda key: int(re.search(r"\.%s:\s+(\d+)" % key, text).group(1))  # noqa: E731
                assert field("private_segment_fixed_size") == 0, "spills"
                found.append(Kernel(m.group(1) == "few", int(m.group(2)), m.group(3) != "f", int(m.group(4)),
                                    int(m.group(5).replace("n", "-")), field("group_segment_fixed_size"), field("vgpr_count"),
                                    field("sgpr_count"), {"f": "f32", "t": "bf16"}.get(m.group(3), "f16")))
        at += 24
    assert len(found) > 100
    return found


def test_caps_hold_for_every_kernel(ask, kernels):
    """At most the workgroups asked for fit into a compute unit with the LDS the kernel really has, and as many as the
    grain of 1280 bytes allows."""
    caps = list(range(2, 32))
    answers = iter(ask([f"lds {k.kind} {int(k.few)} {k.form} {n}" for k in kernels for n in caps]))
    for k in kernels:
        for n in caps:
            own, extra = next(answers)
            assert own <= k.lds <= own + 64, k
            grains = -(-(k.lds + extra) // LDS_GRAIN)
            assert CU_LDS // (grains * LDS_GRAIN) <= n, (k, n)
            assert CU_LDS // ((grains - 1) * LDS_GRAIN) > n or n == 2, (k, n)


def test_sixteen_bit_pipeline_of_single_tiles_keeps_its_wave_slots(kernels):
    """Single tiles of 16-bit gradients run uncapped because they need every wavefront a compute unit can hold: eight per
    SIMD (512 registers, granted in eights), six with the addresses of 16 workers, and no LDS for joined steps."""
    single = [k for k in kernels if KINDS[k.kind] == "pipeline" and k.half and k.form == 1]
    assert len(single) == 20
    for k in single:
        assert 512 // (-(-k.vgprs // 8) * 8) >= (6 if k.P == 16 else 8), k
        assert k.lds <= (0 if k.few else 1296), k


def shapes(ask, cases):
    """launch_shape of each case: a dict of what differs from an even f32 pipeline of 8 workers at the defaults."""
    lines = []
    for c in cases:
        c = dict(kind="pipeline", dtype="f32", P=8, tiles=65536, ragged=0.0, off_lines=0.0, reduced=1, resident=0.0, segments=9,
                 blocks_per_cu=0, xcd_contiguous=0, tiles_per_wg=0, wg_per_cu=0, step_vecs=0, burst_tiles=-1,
                 resident_bytes=0, n_cu=256) | c
        lines.append("shape %d %d %d %d %r %r %d %r %d %d %d %d %d %d %d %d %d" % (
            KINDS.index(c["kind"]), DTYPES.index(c["dtype"]), c["P"], c["tiles"], c["ragged"], c["off_lines"], c["reduced"],
            c["resident"], c["segments"], c["blocks_per_cu"], c["xcd_contiguous"], c["tiles_per_wg"], c["wg_per_cu"], c["step_vecs"],
            c["burst_tiles"], c["resident_bytes"], c["n_cu"]))
    return [Shape(*x) for x in ask(lines)]


PAIRS, BURST, SINGLE = -1, 0, 1


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_pairs_and_their_cap_go_together(ask, dtype):
    """A 16-bit pipeline is capped where its workgroups take pairs of tiles, and nowhere else."""
    def of(**c):
        return shapes(ask, [dict(dtype=dtype, **c)])[0]
    long = of()
    assert (long.form, long.tiles_per_wg, long.wgs_per_cu) == (PAIRS, 2, 14)
    assert of(tiles=1 << 18).wgs_per_cu == 12 and of(tiles=1 << 18, reduced=0).wgs_per_cu == 14
    for single in (of(tiles_per_wg=1), of(resident=0.2, resident_bytes=1 << 20), of(P=2), of(tiles=16383), of(ragged=0.03)):
        assert (single.form, single.tiles_per_wg, single.wgs_per_cu) == (SINGLE, 1, -1)
    for burst in (of(step_vecs=-1), of(burst_tiles=1 << 20), of(tiles=3072), of(step_vecs=-1, tiles_per_wg=2)):
        assert (burst.form, burst.wgs_per_cu) == (BURST, -1)
    assert of(step_vecs=-1).units == 65536                    # and one tile per workgroup
    few = of(resident=0.1, resident_bytes=1 << 20)
    assert (few.form, few.wgs_per_cu) == (PAIRS, 14)
    asked = of(tiles_per_wg=2, P=2)
    assert (asked.form, asked.wgs_per_cu) == (PAIRS, 14)
    asked = of(tiles_per_wg=3, tiles=9000)                    # too short for a cap: every workgroup fits
    assert (asked.form, asked.units, asked.wgs_per_cu) == (PAIRS, 3000, -1)
    assert of(wg_per_cu=21).wgs_per_cu == 21 and of(resident=0.2, wg_per_cu=21).wgs_per_cu == 21
    assert [of(tiles=t).wgs_per_cu for t in (16384, 16500, 17000, 20000, 32767, 32768)] == [16, 18, 18, 14, 16, 14]     # rounds
    for P in (3, 6, 12, 32, 64):                              # not compiled: a ragged tile keeps short launches from pairing
        assert of(P=P, tiles=16384).form == PAIRS and of(P=P, tiles=32767, ragged=1e-5).form == SINGLE
        assert of(P=P, tiles=32768, ragged=0.02).form == PAIRS
    for P in (4, 8, 16):
        assert of(P=P, tiles=16384, ragged=0.02).form == PAIRS
    assert of(P=16, tiles=16500, segments=1).wgs_per_cu == 14                         # registers for 16
    for kind in KINDS:
        if kind != "pipeline":
            assert of(kind=kind).form == SINGLE and of(kind=kind, tiles_per_wg=2).form == SINGLE
    assert shapes(ask, [dict(tiles_per_wg=2)])[0].form == SINGLE


@pytest.mark.parametrize("kind,P,long", [("pipeline", 8, 14), ("reduce", 16, 14), ("direct", 16, 14), ("reduce_update", 32, 14), ("direct", 12, 14),
                                         ("pipeline", 4, 18), ("reduce", 4, 16), ("direct", 8, 16)])
def test_short_binary32_launches_fill_their_rounds(ask, kind, P, long):
    """From the burst form up to 49151 tiles, less with many workers, no neighbour of the cap taken would have fuller rounds, and a launch that
    fits at once runs at once; longer ones keep the cap of long launches."""
    end = min(49152, -(-500000 // P))
    tiles = list(range(3073, end, 97)) + [4096, 5120, 5121, 6400, 6401, 7168, 8192, end - 1]
    got = shapes(ask, [dict(kind=kind, P=P, tiles=t) for t in tiles])
    limited = P == 16 and kind != "reduce"                                        # 16 workers: registers for 16
    near = (18, 21) if long != 14 else (14, 16) if limited else (14, 16, 18)
    for t, s in zip(tiles, got):
        per_cu = -(-t // 256)
        if per_cu <= (16 if limited else 25):
            assert s.wgs_per_cu == 25, t
        else:
            assert s.wgs_per_cu in near, t
            assert -(-per_cu // s.wgs_per_cu) * s.wgs_per_cu == min(-(-per_cu // n) * n for n in near), t
    assert {s.wgs_per_cu for s in shapes(ask, [dict(kind=kind, P=P, tiles=t) for t in (end, 1 << 20)])} == {long}
    assert shapes(ask, [dict(kind=kind, P=P, tiles=6000, n_cu=0)]) == shapes(ask, [dict(kind=kind, P=P, tiles=6000)])
    assert shapes(ask, [dict(kind=kind, P=P, tiles=6000, wg_per_cu=11)])[0].wgs_per_cu == 11
    for few in ("reduce", "reduce_update", "direct"):              # few workers: the cap of long launches at any length
        assert shapes(ask, [dict(kind=few, P=3, tiles=9000)])[0].wgs_per_cu == (-1 if few == "reduce" else 25)


def test_few_segments_form_where_it_pays(ask):
    """The few-segments form is left to the launches it is no slower for: not reductions and single 16-bit tensors
    longer than it pays, and never more segments than the arguments hold."""
    def few(**c):
        return bool(shapes(ask, [dict(segments=1) | c])[0].may_be_few)
    for dtype in DTYPES:
        for P in (1, 3, 8):
            assert few(kind="reduce", tiles=2048, dtype=dtype, P=P, segments=40)       # its segments are groups
            assert not few(kind="reduce", tiles=2049, dtype=dtype, P=P)
    for kind in ("update", "reduce_update", "pipeline", "direct"):
        assert all(few(kind=kind, tiles=t) for t in (1, 3072, 3073, 1 << 20))
        assert few(kind=kind, tiles=100, segments=8) and not few(kind=kind, tiles=100, segments=9)
        assert not few(kind=kind, tiles=100, resident_bytes=8) and not few(kind=kind, tiles=1000, xcd_contiguous=1)
        for dtype in ("bf16", "f16"):
            per_wg = dict(tiles_per_wg=1)
            assert all(few(kind=kind, dtype=dtype, tiles=t, **per_wg) for t in (1, 3072, 6145, 8192, 12289, 14336))
            assert not any(few(kind=kind, dtype=dtype, tiles=t, **per_wg) for t in (3073, 6144, 8193, 12288, 14337, 1 << 20))
            assert all(few(kind=kind, dtype=dtype, tiles=t, segments=2) for t in (3073, 6144, 8193, 1 << 20))
    assert few(kind="pack", tiles=1 << 20) and few(kind="pack", dtype="bf16", tiles=512) and few(kind="pack", dtype="bf16", tiles=8193)
    assert not few(kind="pack", dtype="bf16", tiles=513) and not few(kind="pack", dtype="bf16", tiles=8192)
    assert few(kind="pack", dtype="bf16", tiles=513, segments=2)
    # with 16 workers the table form runs 16 tiles per compute unit at once, the few-segments form 20
    caps = shapes(ask, [dict(P=16, tiles=t, segments=n) for t, n in ((4096, 9), (4097, 9), (5120, 1), (5121, 1))])
    assert [s.wgs_per_cu for s in caps] == [25, 14, 25, 14]


def test_shares_are_of_the_launch_and_not_of_the_model(ask):
    """Ragged tiles and tensors off their lines are counted over the groups a call covers: against the tile table and
    the layout for random models, and for an even group beside a thousand odd tensors."""
    rng = np.random.default_rng(1912)
    lines, want = [], []
    models = [([256 * 40000] + [301] * 1000, [0, 0] + [1] * 999)]
    for _ in range(60):
        L = int(rng.integers(1, 40))
        unit = int(rng.choice([1, 1, 32]))
        models.append(([int(x) // unit * unit for x in np.exp(rng.uniform(0, 9, L)) * (rng.random(L) > 0.1)],
                       [0] + [int(x) for x in rng.random(L - 1) < 0.6]))
    for n, merged in models:
        ctx = M.Context(n, merged, 2, M.F32, host_only=True)
        tables = ctx.tables()
        tiles, group_tile = tables["tiles"], tables["group_tile"]
        off, group, _, _ = ctx.layout()
        G = ctx.n_groups
        for g0, g1 in [(0, G), (0, 1), (G - 1, G), tuple(sorted(int(x) for x in rng.integers(0, G + 1, 2)))]:
            part = tiles[group_tile[g0]:group_tile[g1]]
            if len(part) == 0:
                continue
            elems = [(n[i], (n[i] | int(off[i])) % 32 != 0) for i in range(len(n)) if g0 <= group[i] < g1]
            lines.append("shares %d %s %d %d" % (len(n), " ".join(f"{x} {m}" for x, m in zip(n, merged)), g0, g1))
            want.append((len(part), int(((part["nseg"] > 1) | (part["valid"] < 256)).sum()),
                         round(1e6 * sum(x for x, o in elems if o) / sum(x for x, _ in elems))))
        ctx.close()
    assert ask(lines) == want
    assert want[1] == (1176, 997, 1000000) and want[2] == (40000, 0, 0)      # the odd tensors first, the even group last


def test_ragged_launches_run_uncapped_where_that_helps(ask):
    for kind in ("pipeline", "reduce_update", "direct"):
        caps = shapes(ask, [dict(kind=kind, P=P, ragged=r) for P in (3, 6, 12, 32, 4, 8, 16) for r in (0.2, 0.3)])
        assert all(a.wgs_per_cu > 0 for a in caps[::2]) and all(b.wgs_per_cu == -1 for b in caps[1:10:2])
        assert [b.wgs_per_cu for b in caps[11::2]] == [a.wgs_per_cu for a in caps[10::2]]     # 8 and 16 workers
    assert shapes(ask, [dict(kind="reduce", P=6, ragged=0.9)])[0].wgs_per_cu == 16            # nothing ragged about it


def test_shares_of_sixteen_bit_packs(ask):
    """Eight tiles per workgroup at a cap of 21 in the longest even launches of many workers only."""
    def share(**c):
        s = shapes(ask, [dict(kind="pack", dtype="bf16") | c])[0]
        return s.tiles_per_wg, s.wgs_per_cu
    assert share(P=32, tiles=99832, ragged=0.00017) == (8, 21) and share(P=12, tiles=87400) == (8, 21)
    for c in (dict(P=8, tiles=200000), dict(P=12, tiles=87000), dict(P=32, tiles=32768), dict(P=32, tiles=99832, ragged=0.0005)):
        assert share(**c) == (4, -1), c
    assert share(P=8, tiles=8192) == (2, -1) and share(P=2, tiles=1024) == (1, -1)


def test_runs_per_die_where_they_help(ask):
    def run(kind, P, off, dtype="f32", **c):
        return shapes(ask, [dict(kind=kind, P=P, off_lines=off, dtype=dtype) | c])[0].run_log2
    assert [run(k, 3, 0.26) for k in KINDS] == [0, 0, 3, 3, 2, 3] and not any(run(k, 3, 0.25) for k in KINDS)
    assert [run(k, 8, 0.5) for k in KINDS] == [0, 0, 3, 0, 2, 0] and [run(k, 8, 0.51) for k in KINDS] == [0, 0, 3, 3, 2, 3]
    assert [run(k, 12, 1.0) for k in KINDS] == [0, 0, 3, 0, 2, 3]          # reduce_update of many workers: never
    assert [run(k, 16, 0.26, "bf16") for k in KINDS] == [0, 0, 3, 3, 2, 3] and run("reduce_update", 24, 1.0, "bf16") == 0
    assert run("update", 1, 1.0, xcd_contiguous=1) == 0 and run("update", 1, 1.0, blocks_per_cu=4) == 0


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not available")
def test_builds_with_other_tiles_compile():
    """What a tuning build may override (build_library's `defines`): every kernel is instantiated, none compiled."""
    from paper_1912_09268_amd import build as B
    runs = [subprocess.Popen(["hipcc", *B.HIPCC_FLAGS, "-w", *(f"-D{d}" for d in defines), "-I", os.path.join(ROOT, "include"),
                              "-I", CSRC, "-x", "hip", "-fsyntax-only", os.path.join(CSRC, "kernels.hip")],
                             stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
            for defines in (["MGWFBP_TILE_VECS=2"], ["MGWFBP_TILE_VECS=4", "MGWFBP_PACK_TILES=1"], ["MGWFBP_BLOCK=128"],
                            ["MGWFBP_BLOCK=256", "MGWFBP_TILE_VECS=2", "MGWFBP_PACK_TILES=4"])]
    for run in runs:
        out = run.communicate(timeout=120)[0]
        assert run.returncode == 0, out


def test_binary32_pipelines_without_the_reduced_arena_take_a_wider_window(ask):
    for P, with_it, without in ((4, 18, 18), (6, 14, 16), (8, 14, 16), (12, 14, 16), (16, 14, 14), (32, 14, 14)):
        long = shapes(ask, [dict(P=P, tiles=99832, reduced=r) for r in (1, 0)])
        assert [s.wgs_per_cu for s in long] == [with_it, without], P
        short = shapes(ask, [dict(P=P, tiles=t, reduced=r) for t in range(3073, 30000, 311) for r in (1, 0)])
        assert short[::2] == short[1::2]                     # where the rounds decide they decide alike


def test_burst_form_ends_where_pacing_is_ahead(ask):
    """The longest launch in the burst form by kind, gradient width and worker count."""
    for kind, dtype, P, tiles in (("pipeline", "f32", 3, 3072), ("pipeline", "f32", 8, 1792), ("pipeline", "f32", 16, 1280), ("pipeline", "bf16", 16, 3072),
                                  ("reduce", "f32", 5, 1792), ("reduce", "f32", 6, 1792), ("reduce", "f32", 32, 1792), ("reduce", "f32", 8, 1280), ("reduce", "f32", 16, 1280),
                                  ("reduce_update", "f32", 8, 1792), ("reduce_update", "f32", 16, 1536), ("direct", "f32", 4, 2560), ("direct", "f32", 16, 1792), ("direct", "f16", 8, 3072),
                                  ("update", "f32", 8, 3072)):
        assert [s.form for s in shapes(ask, [dict(kind=kind, dtype=dtype, P=P, tiles=t) for t in (1, tiles, tiles + 1)])] == [BURST, BURST, SINGLE], (kind, P)


def test_long_sixteen_bit_reduce_update_is_capped(ask):
    """Capped from twice SHORT_LAUNCH_TILES on with 4 to 16 workers; every wave slot otherwise."""
    def cap(P, tiles, dtype="bf16"):
        return shapes(ask, [dict(kind="reduce_update", dtype=dtype, P=P, tiles=tiles)])[0].wgs_per_cu
    for dtype in ("bf16", "f16"):
        assert [cap(P, 32768, dtype) for P in (1, 3, 4, 12, 16, 17, 32)] == [-1, -1, 25, 25, 25, -1, -1]
        assert [cap(P, 32767, dtype) for P in (4, 16)] == [-1, -1]


@pytest.mark.parametrize("block,tile_vecs", [(64, 1), (64, 2), (128, 1), (128, 2), (256, 1)])
def test_tiles_go_piece_by_piece_in_workgroups_of_one_wavefront(tmp_path, block, tile_vecs):
    """The last vector of a piece shares elements with the one before it, so the lanes that take them (of 257 to 259
    elements lanes 63 and 64) must be of one wavefront: another could update w and v before they are read.  Without the
    pieces reductions have the general path's LDS."""
    ask = build_driver(tmp_path, f"MGWFBP_BLOCK={block}", f"MGWFBP_TILE_VECS={tile_vecs}")
    (pairs, few, pieces), = ask(["have"])
    assert (pairs, few, pieces) == (tile_vecs == 1, tile_vecs == 1 and block == 64, tile_vecs == 1 and block == 64)
    (own, _), = ask(["lds %d 0 1 0" % KINDS.index("reduce")])
    assert own == (0 if pieces else 4 * (block * tile_vecs + 1))


def wavefronts(k):
    """That a compute unit holds of a kernel, by its registers: a SIMD has 512 vector registers, granted in eights, and 800
    scalar ones, granted in sixteens, of which every wavefront takes one block more than it asks for."""
    return 4 * min(8, 512 // (-(-k.vgprs // 8) * 8), 800 // (-(-k.sgprs // 16) * 16 + 16))


def test_few_segments_kernels_of_sixteen_bit_gradients_keep_their_wave_slots(kernels):
    """Launches over one 16-bit tensor of 25 to 32 tiles per compute unit take the few-segments form because they fit at once
    in it: scalar registers, above all, must not keep them from that."""
    least = {"direct": {}, "update": {}, "reduce_update": {}, "pipeline": {8: 28, 16: 24}}
    paced = [k for k in kernels if k.few and k.half and k.form == 1 and KINDS[k.kind] in least]
    assert len(paced) == 2 * (1 + 3 * 5)
    for k in paced:
        assert wavefronts(k) >= least[KINDS[k.kind]].get(k.P, 32), k


def test_general_path_where_pieces_cost_wavefronts(kernels):
    """Paced 16-bit steps of reduce_update leave ragged tiles of several tensors to the general path with 8 and 16 workers."""
    of = {(k.dtype, k.P): wavefronts(k) for k in kernels if KINDS[k.kind] == "reduce_update" and k.form == 1 and not k.few}
    assert of["bf16", 8] == 32 and of["bf16", 16] == 28 and of["f16", 8] == 28


def per_cu(*counts):
    return [int(256 * c) for c in counts]


def test_pipeline_rolls_where_that_is_no_slower(ask, kernels):
    """Both sides of every line: binary32 up to 12 tiles per compute unit, 11 with 8 and 16 workers, 10 over many tensors where
    the worker count is not compiled; 16-bit gradients up to 16, and up to 36 where the kernel cannot hold them all at once;
    never beside a caller's pacing, nor in the burst form or in pairs, nor in another kind."""
    def rolls(counts, segments, **c):
        return [bool(s.rolling) for s in shapes(ask, [dict(tiles=t, segments=segments, burst_tiles=0) | c for t in per_cu(*counts)])]
    for P in (1, 2, 3, 4, 8, 12, 16, 32):
        last = {8: (11, 11), 16: (11, 11), 2: (12, 12), 4: (12, 12)}.get(P, (12, 10))
        held = {2: (32, 28), 4: (32, 24), 8: (28, 24), 16: (24, 24)}.get(P, (32, 32))
        for segments, end, at_once in zip((8, 9), last, held):
            assert rolls(range(1, 31), segments, P=P) == [n <= end for n in range(1, 31)], (P, segments)
            for dtype in ("bf16", "f16"):
                counts = range(1, 60)
                assert rolls(counts, segments, P=P, dtype=dtype) == [n <= 16 or at_once < n <= 36 for n in counts], (P, segments)
    for off in (dict(wg_per_cu=25), dict(wg_per_cu=-1), dict(step_vecs=1), dict(step_vecs=-1), dict(burst_tiles=1 << 20), dict(kind="direct"),
                dict(kind="pack"), dict(dtype="bf16", tiles_per_wg=2)):
        assert not any(rolls((4, 12), 9, **off)), off
    # the wavefronts that the lines of 16-bit gradients rest on
    single = [k for k in kernels if k.half and k.form == 1 and KINDS[k.kind] == "pipeline"]
    for few, held in ((True, {2: 32, 4: 32, 8: 28, 16: 24, 0: 32}), (False, {2: 28, 4: 24, 8: 24, 16: 24, 0: 32})):
        assert {k.P: wavefronts(k) for k in single if k.few == few and k.P in held} == held
    # and the sizes at which the GPU tests run rolling steps and single ones
    assert rolls((2500 / 256, 11, 3000 / 256, 3100 / 256), 1) == rolls((2500 / 256, 11, 3000 / 256, 3100 / 256), 10) == [True, True, False, False]
    assert rolls((2500 / 256, 11, 3000 / 256, 3100 / 256), 1, P=3) == [True, True, True, False] and rolls((2500 / 256, 11), 10, P=3) == [True, False]
    assert [rolls((4000 / 256, 4100 / 256, 6300 / 256, 34), n, dtype="bf16") for n in (1, 10)] == [[True, False, False, True], [True, False, True, True]]


def test_sixteen_bit_launches_of_a_few_rounds_fill_them(ask, kernels):
    """Uncapped 16-bit launches in single tiles are held to 24 wavefronts per compute unit where that takes no more rounds than
    the 32 or 28 their kernel has registers for, and only there."""
    counts = list(range(13, 128))

    def capped(**c):
        got = shapes(ask, [dict(dtype="bf16", tiles=t) | c for t in per_cu(*counts)])
        assert {s.wgs_per_cu for s in got} <= {25, -1} and {s.form for s in got} <= {SINGLE}
        return [n for n, s in zip(counts, got) if s.wgs_per_cu == 25]
    at_32, at_28 = [*range(33, 49), *range(65, 73)], [*range(29, 49), *range(57, 73), *range(85, 97), *range(113, 121)]
    assert capped(kind="direct", segments=9, ragged=0.3) == []                     # ragged launches want every slot
    for segments in (5, 9):
        for P in (1, 2, 3, 4, 8, 12, 16, 32):
            assert capped(kind="direct", P=P, segments=segments) == at_32
            held = at_28 if P == 16 and segments == 9 else at_32
            assert capped(kind="reduce_update", P=P, segments=segments) == held, P
            if P not in (2, 4, 8, 16):
                assert capped(P=P, segments=segments, ragged=0.03) == at_32
            else:
                assert capped(P=P, segments=segments, ragged=0.03) == []
    assert capped(kind="reduce_update", P=8, dtype="f16") == at_28 and capped(kind="update") == [] and capped(kind="direct", wg_per_cu=-1) == []
    slots = {(KINDS[k.kind], k.few, k.P): wavefronts(k) for k in kernels if k.half and k.form == 1}
    assert all(slots["reduce_update", True, P] == 32 for P in (0, 2, 4, 8, 16)) and slots["pipeline", False, 0] == 32


def test_launches_of_mostly_ragged_tiles_go_in_pieces(ask):
    assert [bool(s.in_pieces) for s in shapes(ask, [dict(kind="direct", dtype="bf16", P=16, ragged=r) for r in (0.0, 0.5, 0.51, 1.0)])] == [False, False, True, True]


def test_pack_and_reduce_have_no_kernels_of_another_store_policy(kernels):
    """Both stream what they write at every size, in kernels of the burst form and of paced steps of one vector only."""
    assert {k.form for k in kernels if KINDS[k.kind] == "pack"} == {SINGLE}
    assert {k.form for k in kernels if KINDS[k.kind] == "reduce"} == {BURST, SINGLE}


@pytest.mark.parametrize("line", [32, 64])
def test_shares_that_begin_on_lines_cover_every_element_once(ask, line):
    """Where UPDATE and DIRECT cut the tensors: tensors of one element to several tiles, tiles with many of them, weights at any address.
    Every element belongs to one tile, and every cut inside a tensor lies on a line of its weights."""
    rng = np.random.default_rng(line)
    lines, models = [], []
    for _ in range(60):
        L = int(rng.integers(1, 40))
        n = [int(x) for x in rng.choice([0, 1, 2, 3, 5, 31, 33, 63, 64, 65, 191, 193, 224, 255, 256, 257, 511, 512, 513, 700, 3000], L)]
        weights = [4 * int(x) for x in rng.integers(1 << 20, 1 << 30, L)]
        merged = [0] + [int(x) for x in rng.random(L - 1) < 0.7]
        models.append((n, weights))
        lines.append(f"cuts {line} {L} " + " ".join(f"{a} {m} {w}" for a, m, w in zip(n, merged, weights)))
    for (n, weights), out in zip(models, ask(lines)):
        shares = {i: [] for i in range(len(n))}
        for layer, lo, hi in zip(out[::3], out[1::3], out[2::3]):
            assert lo <= hi
            if lo < hi:
                shares[layer].append((lo, hi))
        for i, size in enumerate(n):
            at = 0
            for lo, hi in shares[i]:                   # in tile order
                assert lo == at
                at = hi
                assert hi == size or (weights[i] // 4 + hi) % line == 0
            assert at == size


def test_shares_begin_on_lines_where_that_pays(ask):
    """Long launches of UPDATE, and of DIRECT without the reduced arena, over models off their lines."""
    def on_lines(kind, dtype, tiles, segments=100, off=0.5, reduced=0):
        return ask([f"on_lines {KINDS.index(kind)} {DTYPES.index(dtype)} {reduced} {tiles} {segments} {off}"])[0][0]
    for kind, dtype, least in (("update", "f32", 24576), ("update", "bf16", 24576), ("direct", "f32", 24576), ("direct", "f16", 16384), ("direct", "bf16", 16384)):
        assert [on_lines(kind, dtype, t) for t in (least - 1, least)] == [0, 1]
        assert [on_lines(kind, dtype, 32000, segments=x) for x in (2000, 2001)] == [1, 0]
        assert [on_lines(kind, dtype, 100000, off=x) for x in (0.25, 0.26)] == [0, 1]
        assert [on_lines(kind, dtype, 100000, segments=x) for x in (1, 8, 9)] == [1, 1, 1]          # in the table form, also where the other could take it
    assert [on_lines("direct", d, 100000, reduced=1) for d in DTYPES] == [0, 0, 0]
    assert [on_lines(k, "f32", 100000) for k in ("pack", "reduce", "reduce_update", "pipeline")] == [0, 0, 0, 0]


def test_runs_per_die_of_launches_that_begin_on_lines(ask):
    """They stay in the longer ones of updates, of direct steps of one binary32 worker and of up to 16 16-bit ones (over few tensors: of
    up to 7 16-bit ones); shorter launches, and those of other kinds and of the table form, are as the rule of runs says."""
    def runs(kind, dtype, P, tiles, **more):
        return [s.run_log2 for s in shapes(ask, [dict(kind=kind, dtype=dtype, P=P, tiles=t, off_lines=0.6, reduced=0) | dict(segments=100) | more for t in tiles])]
    edge, few = [49151, 49152, 1000000], [65535, 65536, 1000000]
    for dtype, P in [("f32", 1)] + [(d, P) for d in ("bf16", "f16") for P in (1, 3, 7, 8, 16)]:
        assert runs("direct", dtype, P, edge) == [0, 3, 3], (dtype, P)
        assert runs("direct", dtype, P, edge, blocks_per_cu=4) == [0, 0, 0]
        assert runs("direct", dtype, P, edge, resident=0.01, resident_bytes=1 << 20) == [0, 0, 0]
        assert runs("direct", dtype, P, few, segments=8) == ([0, 3, 3] if P < 8 and dtype != "f32" else [0, 0, 0]), (dtype, P)
    for dtype, P in (("f32", 2), ("f32", 8), ("bf16", 17), ("f16", 32)):
        assert runs("direct", dtype, P, edge) == [0, 0, 0], (dtype, P)
    for dtype in DTYPES:
        assert runs("update", dtype, 8, [24575, 24576, 49151, 49152, 131072, 131073]) == [3, 0, 0, 3, 3, 0]       # on lines from 24576
        assert runs("update", dtype, 8, few, segments=8) == [0, 0, 0]
    assert runs("pipeline", "f32", 8, edge) == [2, 2, 2]
    assert [runs("direct", "f32", 1, [30000], reduced=r) for r in (0, 1)] == [[0], [3]]


def test_long_binary32_launches_write_through_the_l2(ask):
    """From a quarter of LONG_LAUNCH_TILES on, models on their lines with few ragged tiles, in the table form."""
    def through(kind, dtype="f32", tiles=65536, off=0.0, ragged=0.0, segments=100):
        return ask([f"through {KINDS.index(kind)} {DTYPES.index(dtype)} {tiles} {off} {ragged} {segments}"])[0][0]
    for kind in ("reduce_update", "pipeline", "direct"):
        assert [through(kind, tiles=t) for t in (65535, 65536, 1000000)] == [0, 1, 1]
        assert [through(kind, off=x) for x in (0.25, 0.26)] == [1, 0]
        assert [through(kind, ragged=x) for x in (0.024, 0.025)] == [1, 0]
        assert [through(kind, segments=x) for x in (8, 9)] == [0, 1]
        assert [through(kind, dtype=d) for d in DTYPES] == [1, 0, 0]
    assert [through(k) for k in ("pack", "reduce", "update")] == [0, 0, 0]
