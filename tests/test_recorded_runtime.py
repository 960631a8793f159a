"""Host code of the library on a recording runtime (hip_recorder.c): what it allocates, frees and
launches, without a GPU."""
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.environ.get("FLASHSKETCH_LIB", os.path.join(HERE, "..", "paper_2602_06071_amd", "libflashsketch.so"))


@pytest.fixture(scope="module")
def recorded(tmp_path_factory):
    """Runs Python source with the names of recorded.py in a process of its own."""
    cc = shutil.which("gcc")
    if not cc:
        pytest.skip("no C compiler")
    rec = str(tmp_path_factory.mktemp("recorder") / "recorder.so")
    subprocess.run([cc, "-shared", "-fPIC", "-O1", "-o", rec, os.path.join(HERE, "hip_recorder.c")], check=True)

    def run(source):
        r = subprocess.run([sys.executable, os.path.join(HERE, "recorded.py"), rec, LIB], input=source, text=True,
                           capture_output=True, timeout=120)
        assert r.returncode == 0, r.stderr
        return r.stdout
    return run


def test_a_workspace_that_serves_a_call_is_kept_when_memory_is_short(recorded):
    recorded("""
s = Sketch(262144, 4096, 2048, 32, 4, 4)
rec.rec_budget(8 << 20)                       # no room for the usual first size
assert s.apply_rows(2) == 0                   # input-stationary: it must have one
held = s.info().workspace_bytes
assert 0 < held < (8 << 20) and len(lines("malloc-failed")) == 1
for n in (2, 1):
    rec.rec_clear()
    assert s.apply_rows(n) == 0
    assert not lines("free") and not lines("malloc") and not lines("malloc-failed"), lines()
rec.rec_budget(1 << 40)
rec.rec_clear()
assert s.apply_rows(64) == 0                  # needs more: replaced
assert len(lines("free")) == 1 and s.info().workspace_bytes > held

s = Sketch(16384, 1024, 1024, 64, 4, 8)       # output-stationary: runs without any
rec.rec_budget(rec.rec_live() + (1 << 20))
assert s.apply_rows(4) == 0 and s.info().workspace_bytes == 0
rec.rec_clear()
assert s.apply_rows(4) == 0
assert not lines("malloc-failed"), lines()    # not asked for again on every call
""")


@pytest.mark.parametrize("replace", ["s.apply(512)", "s.attach(1 << 42, 1 << 30)"])
@pytest.mark.parametrize("captured", [True, False])
def test_a_workspace_that_a_graph_uses_outlives_its_replacement(recorded, captured, replace):
    recorded(f"""
captured = {captured}
s = Sketch(262144, 4096, 2048, 32, 4, 4)
assert s.apply_rows(2, stream=STREAM) == 0
address = lines("malloc")[0][0]               # the workspace (then the wiring's table)
rec.rec_capturing(int(captured))
assert s.apply_rows(2, stream=STREAM) == 0
rec.rec_capturing(0)
rec.rec_clear()
assert {replace} == 0                         # a larger one takes its place
assert lines("free") == ([] if captured else [[address]])
rec.rec_clear()
assert s.destroy() == 0
assert ([address] in lines("free")) == captured and rec.rec_live() == 0
""")


def test_the_lds_limit_is_raised_on_every_device(recorded):
    recorded("""
calls = [((4096, 256, 512, 32, 2, 4), 512, F32, "ksplit_kernel"), ((65536, 8192, 64, 8, 8, 2), 300, BF16, "mfma_kernel"),
         ((16384, 1024, 1024, 64, 4, 8), 16384, F32, "stacked_kernel")]
for params, n, dtype, kernel in calls:
    for device in (0, 1, 0, 70):              # each device has limits of its own, whatever its number
        rec.rec_device(device)
        s = Sketch(*params)
        assert s.apply(n, dtype) == 0 and s.kernel().startswith(kernel), s.kernel()
    big = [l for l in launches() if l.lds > 64 * 1024]
    assert {l.device for l in big} == {0, 1, 70}, kernel
    seen = set()
    for ln in lines():
        if ln[0] == "lds-limit":
            seen.add((ln[1], ln[3], int(ln[2])))
        elif ln[0] == "launch" and int(ln[6]) > 64 * 1024:
            assert any(k == ln[1] and dev == ln[7] and limit >= int(ln[6]) for k, dev, limit in seen), ln
    rec.rec_clear()
""")


def test_a_dense_sketch_that_just_fits_is_created_and_does_not_split(recorded):
    recorded("""
k, d, n = 256, 4096, 64
matrix = 14 * k * d                           # fp32 and five 16-bit copies
for room, status, splits in ((matrix + (128 << 20), 0, True), (matrix + (1 << 20), 0, False), (matrix - 1, 3, None)):
    rec.rec_budget(rec.rec_live() + room)
    s = Sketch(d, k, kind=2)
    assert s.status == status, room
    if status == 0:
        rec.rec_clear()
        assert s.apply(n) == 0
        assert ([l.z > 1 for l in launches()] == [splits] + [False] * splits), launches()
        assert s.destroy() == 0
    assert rec.rec_live() == 0
""")


def test_creating_a_dense_sketch_does_not_swallow_an_error_of_the_program(recorded):
    recorded("""
rec.rec_pending(700)
s = Sketch(4096, 256, kind=2)
assert s.status == 4 or rec.hipGetLastError() == 700      # reported, or still there
if s.status:
    assert not s.h.value and rec.rec_live() == 0
rec.rec_budget(rec.rec_live() + (16 << 20))               # out of memory is create's own: it leaves nothing
rec.rec_pending(0)
s = Sketch(4096, 256, kind=2)
assert s.status == 0 and rec.hipGetLastError() == 0
""")


def test_the_kernel_scope_of_a_profile_holds_every_pass_over_the_input(recorded):
    """A larger fp32 call of the dense sketch reads A twice: for the column maxima and for the product."""
    recorded("""
s = Sketch(16384, 2048, kind=2)
assert lib.fs_sketch_profile_begin(s.h, 1, 1) == 0
rec.rec_clear()
assert s.apply(512) == 0
log = [ln[1] if ln[0] == "launch" else ln[0] for ln in lines() if ln[0] in ("launch", "event")]
maxima, product = ([i for i, w in enumerate(log) if name in w] for name in ("gauss_colmax", "gauss_kernel"))
assert len(maxima) == 1 and product, log      # (the half pieces are taken here)
events = [i for i, w in enumerate(log) if w == "event"]
assert len(events) == 2 and events[0] < maxima[0] and max(product) < events[1], log
""")


def test_a_dense_sketch_without_room_for_half_pieces_splits_and_keeps_three(recorded):
    recorded("""
k, d, n = 2816, 4992, 152                     # taken in half pieces where a handle has them
for room, half in ((20 * k * d + (128 << 20), True), (14 * k * d + (65 << 20), False)):
    rec.rec_budget(rec.rec_live() + room)
    s = Sketch(d, k, kind=2)
    assert s.status == 0 and len(lines("malloc-failed")) == (0 if half else 1)
    rec.rec_clear()
    assert s.apply(n) == 0 and (",half," in s.kernel()) == half and s.kernel().endswith("+reduce_planes"), s.kernel()
    assert ("gauss_colmax" in launches()[0].kernel) == half and launches()[-2].z > 1
    assert s.destroy() == 0 and rec.rec_live() == 0
    rec.rec_clear()
""")


@pytest.mark.parametrize("k,d,n,splits", [
    (3200, 37504, 64, 10),    # 25 row tiles: 250 work-groups in one round (20 splits would be two rounds of 30 stages for one of 59)
])
def test_dense_fp32_work_groups_that_fill_the_lds_alone_are_priced_in_whole_rounds(recorded, k, d, n, splits):
    """Three pieces of 128 x 64 of S, twice, are 108 KiB: a CU of 160 KiB holds one such work-group."""
    recorded(f"""
rec.rec_budget(rec.rec_live() + 14 * {k} * {d} + (65 << 20))   # no room for the half pieces
s = Sketch({d}, {k}, kind=2)
rec.rec_clear()
assert s.status == 0 and s.apply({n}) == 0
run = launches()[0]
assert "gauss_kernel" in run.kernel and 2 * run.lds > 160 << 10, run
assert run.x * run.y * run.z <= 256 and run.z == {splits}, run
""")


@pytest.mark.parametrize("k,d,n,dtype,stages", [
    (2048, 47808, 436, "BF16", 47),    # 747 stages for 16 row tiles: 16 splits are one whole round of 256 work-groups
    (3584, 7424, 392, "F16", 17),
])
def test_a_dense_call_is_split_by_whole_stages_odd_or_even(recorded, k, d, n, dtype, stages):
    recorded(f"""
s = Sketch({d}, {k}, kind=2)
rec.rec_clear()
assert s.apply({n}, {dtype}) == 0
run = launches()[0]
assert "gauss_kernel" in run.kernel and "Li4ELi1ELi4E" in run.kernel and run.z == -(-({d} // 64) // {stages}), run
assert "Li4ELi1ELi4ELb0ELb1E" in run.kernel, run      # the variant for an odd number of stages: none is added to a full split
""")


def test_a_dense_call_on_half_pieces_is_followed_by_the_kernel_for_columns_of_few_terms(recorded):
    """(It takes the column tiles that the other left: same grid, same planes.)"""
    recorded("""
for k, d, n, half in ((4096, 4096, 1030, True), (2816, 4992, 152, True), (1664, 44096, 44, True), (384, 4608, 44, False),
                      (4096, 512, 4096, False)):          # (512 rows: a dense column has hardly the terms)
    s = Sketch(d, k, kind=2)
    rec.rec_clear()
    assert s.apply(n, ld=(n + 3) & ~3) == 0
    run = [l for l in launches() if "reduce" not in l.kernel]
    assert len(run) == (3 if half else 1), run
    pieces = [2 if "ELb1ELb" in l.kernel else 3 for l in run if "12gauss_kernel" in l.kernel]
    assert pieces == ([2, 3] if half else [3]), run
    if half:
        assert "gauss_colmax" in run[0].kernel and run[1][1:5] == run[2][1:5], run
    s.destroy()
""")


SPLIT = """
def split(s, n, dtype, ld=None):              # the kernels of a call and their row split
    rec.rec_clear()
    assert s.apply(n, dtype, ld) == 0
    run = [l for l in launches() if "orbit" not in l.kernel]
    return [l.kernel for l in run], run[0].z
"""


def test_a_multiple_of_256_columns_is_planned_like_its_neighbours(recorded):
    recorded(SPLIT + """
for params, n, dtype in [((281454, 1632, 5598, 32, 3, 2), 512, BF16), ((388370, 2464, 5057, 32, 3, 2), 768, BF16),
                         ((37820, 792, 384, 8, 2, 2), 512, BF16), ((102472, 2048, 3264, 64, 2, 2), 512, F16),
                         ((30686, 192, 1313, 8, 8, 2), 768, F32)]:
    assert split(Sketch(*params), n, dtype) == split(Sketch(*params), n - 4, dtype), params
""")


def test_few_blocks_split_a_call_as_its_256_column_chunks(recorded):
    """Up to 8 blocks: same kernels and row split at 256, 512, 768 and 1024 columns, wherever the planes fit
    32 MiB at 1024 columns and the reduction adds them in the same way at all widths."""
    recorded(SPLIT + """
import random
rng, held = random.Random(1), 0
for i in range(600):
    M, Br = rng.randrange(1, 9), rng.choice([1, 4, 6, 8, 16, 32, 64])
    kappa, Bc = rng.randrange(1, M + 1), rng.choice([rng.randrange(1, 29000), 64 * rng.randrange(1, 140)])
    s = Sketch(Bc * M - rng.randrange(Bc), Br * M, Bc, Br, kappa, 1)
    dtype, ld = rng.randrange(3), 1024 + rng.choice([0, 0, 1, 2, 4])
    chunk = split(s, 256, dtype, ld)
    planes = chunk[1] * kappa
    if s.info().last_mode == 2 and planes * s.k * 4096 <= 32 << 20 and (planes < 16 or s.k < 256 or s.k >= 1024):
        held += 1
        for n in (512, 768, 1024):
            assert split(s, n, dtype, ld) == chunk, (s.d, s.k, Bc, Br, kappa, dtype, ld, n)
    s.destroy()
assert held > 300
""")


@pytest.mark.parametrize("params,n,dtype", [
    ((28288, 14144, 128, 64, 3, 2), 448, "F32"),      # 884 work-groups, one per CU, of one stage per wave
    ((2760, 960, 184, 64, 2, 2), 6592, "F32"),
    ((4925, 308, 64, 4, 2, 2), 256, "F32"),
    ((135660, 24704, 704, 128, 4, 2), 394, "F16"),
])
def test_many_short_rounds_of_work_groups_stay_with_one_wave_per_column_tile(recorded, params, n, dtype):
    assert "mfma_kernel" in recorded(f"s = Sketch(*{params}); assert s.apply({n}, {dtype}) == 0; print(s.kernel())")


@pytest.mark.parametrize("params,n,loads", [
    ((89856, 2808, 128, 4, 1, 2), 213, 4),       # one addend
    ((10864, 484, 90, 4, 2, 2), 1024, 4),        # two
    ((65536, 8192, 64, 8, 8, 2), 256, 8),        # eight
])
def test_the_rows_reduction_loads_no_more_than_it_needs_together(recorded, params, n, loads):
    out = recorded(f"s = Sketch(*{params}); assert s.apply_rows({n}, BF16) == 0; print(launches()[-1].kernel)")
    assert f"reduce_rows_kernelItLi4ELi1ELi{loads}E" in out, out


@pytest.mark.parametrize("params,n,dtype,rows,ld,kernel", [
    # columns of a wide matrix: a cache line per element, kappa times on the kernel of a few vectors
    ((4194304, 8192, 4096, 8, 8, 2), 1, "BF16", False, 64, "ksplit_kernel"),
    ((4194304, 8192, 4096, 8, 8, 2), 2, "BF16", False, 1024, "ksplit_kernel"),
    ((4194304, 8192, 4096, 8, 8, 2), 4, "BF16", False, 16, "ksplit_kernel"),
    ((262144, 4096, 2048, 32, 4, 4), 1, "F32", False, 64, "ksplit_kernel"),
    ((262144, 4096, 2048, 32, 4, 4), 2, "F32", False, 4096, "ksplit_kernel"),
    # packed ones
    ((262144, 4096, 2048, 32, 4, 4), 1, "F32", False, 1, "vector_kernel"),
    ((262144, 4096, 2048, 32, 4, 4), 2, "BF16", False, 2, "vector_kernel"),
    ((262144, 4096, 2048, 32, 4, 4), 1, "F32", True, 262144, "vector_kernel"),
    # longer there than on the kernel it would take the place of
    ((861504, 1024, 53888, 64, 1, 2), 2, "F16", True, 861504, "rows_kernel"),
    ((131661, 1024, 1029, 8, 8, 8), 3, "BF16", False, 3, "ksplit_kernel"),
])
def test_a_few_vectors_take_the_kernel_that_is_shorter_by_its_price(recorded, params, n, dtype, rows, ld, kernel):
    out = recorded(f"s = Sketch(*{params}); assert s.apply{'_rows' if rows else ''}({n}, {dtype}, ld={ld}) == 0; print(s.kernel())")
    assert out.startswith(kernel), out


def test_a_few_vectors_are_refused_exactly_where_the_matrix_core_kernels_are(recorded):
    """Attached workspaces of every size around what the calls ask for, on the static scratch array too."""
    recorded("""
refused = accepted = 0
for params in [(15990, 128, 4000, 32, 2, 4), (16000, 256, 4001, 64, 4, 1), (100000, 16, 50000, 8, 2, 8), (262144, 4096, 2048, 32, 4, 4),
               (20480, 512, 640, 16, 16, 3), (66400, 3200, 333, 16, 8, 5), (4194304, 8192, 4096, 8, 8, 2)]:
    for n in (1, 2, 3, 4):
        for dtype in (F32, BF16, F16):
            for size in [256 << i for i in range(0, 18)]:
                got = []
                for variant in (0, 2):
                    s = Sketch(*params)
                    assert lib.fs_sketch_set_variant(s.h, variant) == 0 and s.attach(1 << 42, size) == 0
                    got.append((s.apply(n, dtype), s.apply_rows(n, dtype), s.apply_static(n, dtype)))
                    s.destroy()
                    rec.rec_clear()
                assert got[0] == got[1], (params, n, dtype, size, got)
                refused += got[0][:2].count(3)
                accepted += got[0][:2].count(0)
assert refused > 100 and accepted > 100
""")


ROWS_FORM = """
import re
def form(s, n, dtype, ld=None):               # of a rows call: (stacked rows / 32, examples / 32, mode, splits, waves, chains of the reduction)
    rec.rec_clear()
    assert s.apply_rows(n, dtype, ld=ld) == 0
    run = [l for l in launches() if "orbit" not in l.kernel]
    mt, et, mode = map(int, re.search(r"rows_kernelI\\w+?Li(\\d)ELi(\\d)ELNS0_8RowsModeE(\\d)E", run[0].kernel).groups())
    chains = int(re.search(r"reduce_rows_kernelI\\w+?Li\\dELi(\\d)E", run[1].kernel).group(1)) if len(run) > 1 else 0
    return mt, et, mode, run[0].z, run[0].threads // 64, chains
"""


def test_rows_forms_that_are_taken_by_price_are_no_less_exact_in_fp32(recorded):
    """Against the form of FS_VARIANT_MFMA, by what the two leave to fp32: twelve roundings per stage of a wave at the size of its
    sum (or of the stage, where that is made apart), one per merged record, the reduction's chains."""
    recorded(ROWS_FORM + """
import math, random
rng, moved = random.Random(2), 0
def error(f, Bc, Br, kappa, sk):
    mt, et, mode, z, nw, chains = f
    total = -(-Bc // 64) * (kappa if mode else 1)
    stages, apart = -(-total // (z * nw)), et == 1 and mt < 4
    dense = 1 - (1 - sk / Br) ** 4            # of the groups of four input rows that meet an output row
    e = 2.6 + (5.4 * dense + 0.44 * stages if apart else 5.9 * dense * stages)
    if chains:
        addends = z * (1 if mode else kappa)
        e += 0.1 + (1.0 if nw > 1 else 0) + (2.4 + 1.25 * addends / 16 if chains > 1 else 0)
    return e / 0.95 if apart else e
cases = [(23637, 4096, 185, 32, 4, 4, 156), (88448, 8192, 173, 16, 4, 8, 64), (10316, 1024, 645, 64, 1, 8, 198), (8585, 2048, 135, 32, 8, 8, 99)]
for i in range(400):
    M, Br, kappa = rng.choice([16, 32, 64, 128, 256]), rng.choice([8, 16, 32, 64, 128]), rng.choice([1, 2, 4, 8])
    Bc = round(math.exp(rng.uniform(math.log(64), math.log(20000))))
    cases.append((Bc * M - rng.randrange(Bc), Br * M, Bc, Br, kappa, rng.choice([2, 4, 8]), round(math.exp(rng.uniform(math.log(33), math.log(1024))))))
for d, k, Bc, Br, kappa, sk, n in cases:
    s = Sketch(d, k, Bc, Br, kappa, sk)
    new = form(s, n, F32)
    assert lib.fs_sketch_set_variant(s.h, 2) == 0
    old = form(s, n, F32)
    s.destroy()
    moved += new != old
    assert error(new, Bc, Br, kappa, sk) <= error(old, Bc, Br, kappa, sk) * 1.0001, (d, k, Bc, Br, kappa, sk, n, old, new)
assert moved > 100
""")


@pytest.mark.parametrize("params,n,dtype,pad", [
    # us per call in this form and in the one the models preferred
    ((26348, 4096, 103, 16, 4, 8), 823, "F16", 0),         # 34.7, 42.1: thirteen rounds of waves with one stage each
    ((145573, 8192, 1138, 64, 1, 4), 538, "F16", 64),      # 38.5, 47.4
    ((520256, 1024, 32516, 64, 1, 2), 336, "BF16", 0),     # 111, 134: bound by the stream of G
    ((511868, 1024, 15996, 32, 1, 4), 524, "F16", 0),      # 138, 164
    ((100544, 4096, 786, 32, 2, 4), 528, "F32", 0),        # 60.8, 75.2
    ((1597598, 2048, 49925, 64, 1, 8), 66, "F16", 0),      # 57, 86
])
def test_rows_calls_that_other_forms_would_slow_down_keep_theirs(recorded, params, n, dtype, pad):
    recorded(ROWS_FORM + f"""
s = Sketch(*{params})
new = form(s, {n}, {dtype}, s.d + {pad})
assert lib.fs_sketch_set_variant(s.h, 2) == 0
assert new == form(s, {n}, {dtype}, s.d + {pad}), new
""")


@pytest.mark.parametrize("params,n,dtype,pad,want", [
    ((9486, 2048, 149, 32, 4, 8), 312, "F16", 64, "one launch"),      # 24.6 -> 9.7 us
    ((5696, 1024, 178, 32, 2, 8), 936, "F16", 0, "one launch"),
    ((23132, 4096, 362, 64, 1, 2), 222, "BF16", 0, "one launch"),     # (kappa = 1: stored by tiles of 64 examples)
    ((93968, 8192, 1472, 128, 8, 8), 529, "F16", 0, "one launch"),    # 356 -> 199
    ((1090981, 2048, 68187, 128, 1, 2), 104, "BF16", 0, "two"),       # 79.6 -> 68.1
])
def test_rows_calls_that_other_forms_speed_up_take_them(recorded, params, n, dtype, pad, want):
    recorded(ROWS_FORM + f"""
s = Sketch(*{params})
mt, et, mode, z, nw, chains = form(s, {n}, {dtype}, s.d + {pad})
assert et < 4 and nw > 1 and (chains == 0) == ({want!r} == "one launch"), (mt, et, mode, z, nw, chains)
""")


def test_a_rows_call_reports_the_mode_that_it_was_planned_in(recorded):
    recorded("""
modes = set()
for params, n, dtype in [((9486, 2048, 149, 32, 4, 8), 312, F16), ((4194304, 8192, 4096, 8, 8, 2), 256, BF16), ((20160, 1280, 1008, 64, 1, 8), 129, F32),
                         ((8192, 1024, 512, 64, 4, 8), 200, F32), ((262144, 4096, 2048, 32, 4, 4), 1, F32), ((262144, 4096, 2048, 32, 4, 4), 24, F32),
                         ((256, 384, 64, 96, 2, 4), 70, F32)]:
    s = Sketch(*params)
    mode = C.c_int32()
    assert lib.fs_sketch_plan(s.h, C.c_void_p(1 << 44), C.c_int64(s.d), C.c_int64(n), dtype, 1, None, C.byref(mode), None, None) == 0
    assert s.apply_rows(n, dtype) == 0 and s.info().last_mode == mode.value, (params, n, s.info().last_mode, mode.value)
    modes.add(mode.value)
assert modes == {0, 1, 2}
""")


def test_the_rows_calls_checked_against_the_oracle_take_the_forms_that_they_name(recorded):
    from test_gpu_parity import ROWS_MANY
    cases = [(params, n, pad, dtype, form) for params, n, pad, form32, form16 in ROWS_MANY
             for dtype, form in (("F32", form32), ("BF16", form16), ("F16", form16))]
    recorded(ROWS_FORM + f"""
for params, n, pad, dtype, want in {cases!r}:
    s = Sketch(*params)
    mt, et, mode, z, nw, chains = form(s, n, globals()[dtype], s.d + pad)
    assert f"{{mt}},{{et}},{{['in', 'out', 'outsplit'][mode]}}" == want and (chains == 0) == (mode == 1), (params, n, dtype, mt, et, mode, z, nw)
    assert nw > 1 or et == 4, (params, n, dtype)
    s.destroy()
""")


@pytest.mark.parametrize("params,n,out", [
    ((8296, 1024, 260, 32, 2, 4), 197, True),       # two stages a wave, one before: error 8.54e-8, 8.55e-8
    ((25920, 1024, 832, 32, 2, 4), 312, False),     # four, two before: 1.10e-7, 1.03e-7
    ((31704, 1024, 991, 32, 2, 4), 257, False),
])
def test_wide_fp32_column_calls_are_stored_in_one_launch_only_by_sums_about_as_short(recorded, params, n, out):
    kernel = recorded(f"s = Sketch(*{params}); assert s.apply({n}, F32) == 0; print(s.kernel())").strip()
    assert kernel.startswith("ksplit_kernel<f32,") and (",out," in kernel) == out and kernel.endswith("+reduce_planes") != out, kernel
