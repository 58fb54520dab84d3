"""The library's host path under failures that a GPU does not produce on demand: the library runs in a process of its own on
tests/host/fake_hip.cpp, a HIP runtime that runs nothing, writes down what it is asked for and fails where it is told to."""
import os
import shutil
import subprocess
import sys
import textwrap

import pytest

from gptq_forms import GPTQ_FORMS
from paper_2309_15531_amd import binding as B
from scoring_forms import GRAM_FORMS, SCORING_FORMS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PREAMBLE = """
import ctypes, sys
from ctypes import byref, c_int32, c_int64, c_void_p, c_char_p, c_double
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)      # ahead of the HIP runtime the library is linked with
fake.fake_calls.restype = c_char_p
lib = ctypes.CDLL(sys.argv[2])
lib.adadim_last_error.restype = c_char_p
OK, EHIP, EINVAL = %d, %d, %d
def context(stream=0x1000):
    h = c_void_p()
    assert lib.adadim_create(byref(h), c_void_p(stream)) == OK
    return h
def calls():
    return fake.fake_calls().decode().split("\\n")[:-1]
def launched(name):
    return [c for c in calls() if c.startswith("launch") and name in c]
A = c_void_p(0x10000)                                          # aligned, never dereferenced: nothing runs
def gemv(ctx, out, inn, bits=4):
    return lib.adadim_gemv_ic(ctx, A, A, A, A, c_int64(out), c_int64(inn), bits, 32, A)
""" % (B.OK, B.EHIP, B.EINVAL)


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    if not os.path.exists(B.LIB_PATH):
        from paper_2309_15531_amd.build import build
        build(verbose=False)
    fake = tmp_path_factory.mktemp("fake") / "libfake_hip.so"
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(ROOT, "tests", "host", "fake_hip.cpp"), "-o",
                    str(fake)], check=True)

    def go(body):
        res = subprocess.run([sys.executable, "-c", PREAMBLE + textwrap.dedent(body), str(fake), B.LIB_PATH],
                             capture_output=True, text=True, timeout=120)
        assert res.returncode == 0, res.stdout + res.stderr
        return res.stdout
    return go


def test_a_failed_allocation_fails_no_later_call(run):
    """The runtime keeps the error of a failed allocation until it is asked for; the next call's launches must not report it."""
    run("""
    ctx = context()
    for call in (lambda: gemv(ctx, 4096, 4096), lambda: lib.adadim_select(ctx, A, 2, None, byref(c_int32()))):
        fake.fake_reset()
        fake.fake_fail(b"hipMalloc", 1)
        assert call() == EHIP
        assert call() == OK, lib.adadim_last_error(ctx)
    """)


@pytest.mark.parametrize("what", ["hipMalloc", "gemv_zero"])
def test_gemv_counters_are_cleared_before_their_first_use(run, what):
    """An allocation or the clearing launch fails in the first call; the next one must clear the counters before a kernel counts
    on them (the block that does not find itself last writes nothing, and the call would return OK)."""
    for nth in (1, 2) if what == "hipMalloc" else (1,):
        run(f"""
        ctx = context()
        fake.fake_fail(b"{what}", {nth})
        first = gemv(ctx, 4096, 4096)
        assert first == EHIP or (first == OK and {nth} > 1), first
        assert gemv(ctx, 4096, 4096) == OK, lib.adadim_last_error(ctx)
        assert gemv(ctx, 4096, 4096) == OK
        order = [c.split()[1] for c in calls() if "gemv" in c]
        assert "gemv_zero" in order[0] and sum("gemv_zero" in c for c in order) == 1, order
        assert "gemv_ic_tiles" in order[-1], order
        """)


def test_gemv_counters_after_the_slot_grew_or_was_recorded(run):
    """Whoever grows the slot, and whether the clearing launch ran or was only recorded, the counters are cleared by a launch
    that has run before one that counts on them."""
    run("""
    ctx = context()
    us = c_double()
    assert gemv(ctx, 1024, 1024) == OK
    assert lib.adadim_probe_gemv_read(ctx, A, c_int64(49152), c_int64(12288), 4, byref(us)) == OK   # grows the same scratch
    g = c_void_p()
    assert lib.adadim_capture_begin(ctx) == OK
    assert gemv(ctx, 1024, 1024) == OK
    assert lib.adadim_capture_end(ctx, byref(g)) == OK
    fake.fake_reset()
    assert gemv(ctx, 1024, 1024) == OK                            # the recorded clearing has not run yet
    order = [c.split()[1] for c in calls() if "gemv" in c]
    assert "gemv_zero" in order[0] and "gemv_ic_tiles" in order[1], order
    fake.fake_reset()
    assert gemv(ctx, 1024, 1024) == OK and not launched("gemv_zero")
    lib.adadim_graph_destroy(g)
    """)


def test_gemv_recording_needs_no_larger_scratch_than_partial_sums_by_whole_rounds(run):
    """Whether a product can be recorded after another one has run once: exactly when whole rounds of 64-lane tiles would need
    no more room for their partial sums, whatever form either takes."""
    run("""
    def need(out, inn):
        tiles = (out + 2047) // 2048
        rounds = (tiles + 255) // 256
        return min(max(1, inn // 256), max(1, rounds * 256 // tiles)) * out * 4
    up = lambda n: (n + 255) // 256 * 256
    shapes = [(32, 4), (32, 4096), (1024, 64), (256, 1024), (288, 1100), (4096, 4096), (4096, 11008), (11008, 4096), (16384, 8192),
              (16416, 260), (28672, 4096), (65536, 2048), (88064, 4096), (131072, 512), (151936, 768), (300032, 64)]
    for a in shapes:
        for b in shapes:
            ctx = context()
            assert gemv(ctx, *a) == OK
            assert lib.adadim_capture_begin(ctx) == OK
            rc = gemv(ctx, *b)
            assert (rc == OK) == (need(*b) <= up(need(*a))), (a, b, rc, need(*a), need(*b))
            g = c_void_p()
            assert lib.adadim_capture_end(ctx, byref(g)) == OK
            lib.adadim_graph_destroy(g)
            lib.adadim_destroy(ctx)
    """)


def test_select_without_pinned_memory(run):
    """The host's index passes through pinned memory; where none can be had the call copies it, as it did before it used any,
    and a later call takes the pinned way again."""
    run("""
    ctx = context()
    dev, host = c_int32(7), c_int32(-1)
    fake.fake_fail(b"hipHostMalloc", 1)
    assert lib.adadim_select(ctx, A, 2, byref(dev), byref(host)) == OK, lib.adadim_last_error(ctx)
    assert host.value == 7
    order = [c.split()[0] for c in calls()]
    assert order[-2:] == ["hipMemcpyAsync", "hipStreamSynchronize"], order
    fake.fake_reset()
    assert lib.adadim_select(ctx, A, 2, byref(dev), byref(host)) == OK
    assert host.value == 0 and not any("hipMemcpyAsync" in c for c in calls())     # the fake kernel left nothing there
    lib.adadim_destroy(ctx)
    """)


def test_per_oc_sweep_takes_the_form_that_is_faster(run):
    """Rows per workgroup of the sweep in one launch, or a launch per 128-channel block (0), beside the times (us) that say so.  A size
    stands here with its times if the two forms, or the best and the second best number of rows, were measured at least 1.015 times apart."""
    run("""
    def form(out, inn):
        ctx = context()
        fake.fake_reset()
        rc = lib.adadim_gptq_quantize(ctx, A, c_int64(out), c_int64(inn), 0, 3, 64 if inn % 64 == 0 else inn, A, A, A, A, A, A, None, None, None, None)
        assert rc == OK, lib.adadim_last_error(ctx)
        rows = [c.split()[1] for c in launched("gq_rows")]
        n = {k: len(launched(k)) for k in ("gq_block", "gq_next")}
        blocks = (inn + 127) // 128
        if not rows:
            assert n == {"gq_block": blocks, "gq_next": blocks - 1 if inn > 256 else 0}, n
            return 0
        assert len(rows) == 1 and n == {"gq_block": 0, "gq_next": 0}, (rows, n)
        return int(rows[0].split("gq_rowsILi")[1].split("E")[0])
    for (out, inn), want in {
        # in one launch / a launch per block
        (300, 2048): 4,          # 270 / 1036
        (2048, 2048): 8,         # 419 / 1104
        (3072, 3072): 12,        # 948 / 1728; 16 rows 990
        (4096, 4096): 16,        # 1611 / 2644
        (4096, 11008): 16,       # 9992 / 12040
        (4608, 4096): 24,        # 2538 / 2868
        (8192, 1024): 32,        # 304 / 616
        (8192, 256): 32,         # 64 / 125
        (6676, 384): 32,         # 96 / 212
        (12288, 6144): 16,       # 10020 / 10620
        (1024, 16384): 4,        # 8539 / 10670
        (16384, 2159): 32,       # 1967 / 2797
        (40000, 1000): 32,       # 1481 / 1999
        (100000, 256): 32,       # 615 / 803
        (28672, 1024): 32,       # 1163 / 1411
        (20000, 256): 32,        # 157 / 236
        (12288, 384): 24,        # 163 / 225; 16 rows 167
        (9216, 4096): 0,         # 4588 / 4305
        (8300, 3300): 0,         # 3230 / 3130
        (8704, 8192): 0,         # 15910 / 13220
        (5632, 11008): 0,        # 16860 / 15270
        (256, 28672): 0,         # 20510 / 16470
        (8, 16384): 0,           # 9868 / 8650
    }.items():
        assert form(out, inn) == want, (out, inn, form(out, inn))
    # channels that are no multiple of four, which the launches per block store element by element, and narrow last blocks
    for shape in ((8192, 131), (7280, 493), (40000, 1533), (8192, 260), (7168, 320), (8192, 200), (7680, 448), (28672, 3003)):
        assert form(*shape) == 32, shape
    for shape, rows in (((64, 2048), 4), ((3072, 128), 12), ((16384, 8192), 32), ((9216, 493), 24), ((9216, 260), 12)):
        assert form(*shape) == rows, shape
    # the sizes whose tests on the GPU aim at a form
    for (out, inn), want in FORMS.items():
        assert form(out, inn) == want, (out, inn, form(out, inn))
    """.replace("FORMS", repr(GPTQ_FORMS)))


def test_narrow_updates_keep_every_wave_busy(run):
    """The update behind a block of the per-OC sweep's launches per block: up to 64 columns the four waves share the rows, beyond
    that the columns (two or three of them had none, and sweeps of 129 to 192 channels, which took this form then, took up to 1.03 times as
    long as with vector instructions)."""
    run("""
    def forms(out, inn):
        ctx = context()
        fake.fake_reset()
        assert lib.adadim_gptq_quantize(ctx, A, c_int64(out), c_int64(inn), 0, 3, inn, A, A, A, A, A, A, None, None, None, None) == OK
        assert launched("gq_block")
        return ["ILb1E" in c for c in launched("gq_trailing")]
    for inn, last in ((3201, True), (3249, True), (3264, True), (3265, False), (3300, False)):
        got = forms(8300, inn)
        assert got == [False] * (len(got) - 1) + [last] and len(got) == 24, (inn, got)
    """)


def test_packers_by_alignment(run):
    """The packers that read several codes at a time serve the widths and addresses that allow it, a thread per word the others
    (byte loads in the tiled packer took up to 2.6 times as long)."""
    run("""
    f1 = ctypes.c_float(1.0)
    def pack(out, inn, dim, codes):
        ctx = context()
        fake.fake_reset()
        assert lib.adadim_quantize(ctx, A, c_int64(out), c_int64(inn), dim, 5, 0, f1, codes, A, A, None, 0, None, A) == OK
        return [c.split()[1] for c in launched("pack_")]
    odd8 = c_void_p(0x10008)
    for out, inn, dim, codes, want in ((513, 4100, 1, A, "pack_wordsILb1E"), (513, 4101, 1, A, "pack_wordsILb1E"),
                                       (513, 4104, 1, A, "pack_columnsILi5ELb0E"), (513, 4112, 1, A, "pack_columnsILi5ELb1E"),
                                       (513, 4112, 1, odd8, "pack_columnsILi5ELb0E"), (513, 4096, 0, A, "pack_rows"),
                                       (513, 4096, 0, odd8, "pack_wordsILb0E"), (513, 4100, 0, A, "pack_wordsILb0E")):
        got = pack(out, inn, dim, codes)
        assert len(got) == 1 and want in got[0], (out, inn, dim, got)
    """)


def test_permuting_copies_by_alignment(run):
    """Rows share a workgroup in the copy before the sweep at any alignment (a row each took up to twice as long), in the copy
    after it where several channels are read at a time or a short row leaves threads idle (else sharing took up to 1.4 times as
    long)."""
    run("""
    def copies(out, inn):
        ctx = context()
        fake.fake_reset()
        assert lib.adadim_gptq_quantize(ctx, A, c_int64(out), c_int64(inn), 1, 3, 64, A, A, A, None, None, A, A, A, None, None) == OK
        return [(c.split()[1], int(c.split()[2])) for c in launched("gq_gather_w") + launched("gq_scatter")]
    for out, inn, share in ((4096, 4090, 4), (4096, 513, 4), (2048, 9999, 2), (1024, 514, 1)):
        (k0, n0), (k1, n1) = copies(out, inn)
        assert "ILb0E" in k0 and n0 == out // share, (k0, n0)
        assert "ILb1ELb0E" in k1 and n1 == out, (k1, n1)
    for out, inn in ((8192, 514), (16384, 259)):
        (k1, n1) = copies(out, inn)[1]
        assert "ILb1ELb0E" in k1 and n1 == out // 4, (k1, n1)
    (k0, n0), (k1, n1) = copies(4096, 4096)
    assert "ILb1E" in k0 and n0 == 1024 and "ILb1ELb1E" in k1 and n1 == 1024
    (k0, n0), (k1, n1) = copies(8192, 65)
    assert "ILb0E" in k0 and n0 == 2048 and "ILb1ELb0E" in k1 and n1 == 2048
    """)


def test_per_ic_sweep_is_one_launch_per_block(run):
    """Walks and update of a block are one launch of at most a workgroup per compute unit, however many groups there are, and nothing
    goes to another stream.  (Launches of their own beyond 160 groups, walks by four waves and the update beside them on a side
    stream, took 1.03 to 1.28 times as long at 50 sizes from 161 to 2000 groups.)"""
    run("""
    for groups, group, inn in ((64, 64, 1024), (86, 128, 4096), (165, 64, 1000), (172, 64, 4096), (300, 128, 260), (300, 64, 128), (2000, 64, 512)):
        ctx = context()
        fake.fake_reset()
        assert lib.adadim_gptq_quantize(ctx, A, c_int64(groups * group), c_int64(inn), 1, 3, group, A, A, A, None, None, A, A, A, None, None) == OK
        steps = [c.split() for c in launched("gq_group")]
        assert len(steps) == (inn + 127) // 128 and {s[4] for s in steps} == {"512"}, (groups, group, inn, steps)
        assert all(int(s[2]) <= 256 for s in steps) and not launched("gq_next") and not launched("gq_trailing")
        assert "hipStreamCreateWithFlags" not in calls()
    """)


def test_factor_stays_on_its_stream(run):
    """The factor's launches all go to the context's stream.  A process has four hardware queues: with the update and the inverse on
    streams of their own, two of the three shared a queue as soon as the process used two or three others, and 4096 channels
    took 3100 to 3220 us instead of 2210."""
    run("""
    for n in (64, 1000, 1025, 4096, 8192):
        ctx = context()
        fake.fake_reset()
        assert lib.adadim_gptq_prepare(ctx, A, c_int64(n), ctypes.c_float(0.01), 1, A, A, A) == OK, lib.adadim_last_error(ctx)
        assert launched("chol_diag_inv") and "hipStreamCreateWithFlags" not in calls(), n
    """)


def test_factor_needs_two_matrices_of_scratch(run):
    """Beside the two fp64 matrices the factor allocates a few MiB, whatever its width (the doubling's products are kept for one
    panel; for the whole matrix they were an eighth to a half of the two, which nothing read).  A factor can be recorded
    after one of at least its width has run."""
    run("""
    def factor(ctx, n):
        return lib.adadim_gptq_prepare(ctx, A, c_int64(n), ctypes.c_float(0.01), 1, A, A, A)
    for n in (64, 1000, 1024, 1025, 5000, 8192):
        ctx = context()
        fake.fake_reset()
        assert factor(ctx, n) == OK, lib.adadim_last_error(ctx)
        sizes = sorted(int(c.split()[1]) for c in calls() if c.startswith("hipMalloc "))
        for _ in "AM":
            sizes.remove((8 * n * n + 255) // 256 * 256)
        assert sum(sizes) < 4 << 20, (n, sizes)
        lib.adadim_destroy(ctx)
    for warm in (64, 512, 1024, 1100, 3000):
        for call in (1, 64, 65, 512, 1000, 1024, 1025, 1100, 2900, 3000, 3100):
            ctx = context()
            assert factor(ctx, warm) == OK
            assert lib.adadim_capture_begin(ctx) == OK
            rc = factor(ctx, call)
            assert (rc == OK) == (call <= warm), (warm, call, rc)
            g = c_void_p()
            assert lib.adadim_capture_end(ctx, byref(g)) == OK
            lib.adadim_graph_destroy(g)
            lib.adadim_destroy(ctx)
    """)


def test_sweep_recording_depends_on_sizes_alone(run):
    """A sweep can be recorded after one of at least its size has run, whichever dimension or form either takes."""
    run("""
    def sweep(ctx, out, inn, dim):
        tail = (A, A, A, None, None, None, None) if dim == 0 else (None, None, A, A, A, None, None)
        return lib.adadim_gptq_quantize(ctx, A, c_int64(out), c_int64(inn), dim, 3, 64, A, A, A, *tail)
    by_block = []
    for warm in ((16384, 4096, 0), (16384, 4096, 1), (100032, 512, 0), (4096, 4096, 0), (9024, 4096, 0)):
        for call in ((9216, 512, 0), (4096, 4096, 0), (4096, 4096, 1), (100032, 128, 0), (300, 8192, 0), (8320, 3328, 0)):
            ctx = context()
            assert sweep(ctx, *warm) == OK
            assert lib.adadim_capture_begin(ctx) == OK
            fake.fake_reset()
            rc = sweep(ctx, *call)
            by_block.append(bool(launched("gq_block")))
            assert (rc == OK) == (call[0] * call[1] <= warm[0] * warm[1] and call[1] <= warm[1]), (warm, call, rc)
            g = c_void_p()
            assert lib.adadim_capture_end(ctx, byref(g)) == OK
            lib.adadim_graph_destroy(g)
            lib.adadim_destroy(ctx)
    assert any(by_block) and not all(by_block)                    # both forms
    """)


def test_scoring_and_gram_sizes_take_the_tiles_their_tests_name(run):
    """The edge of the scoring tiles, the chunk of the contraction and the slots of each size in the tests' table, whichever entry point and input
    it comes by; and the edge of the Gram matrix's tiles.  (Lines between the kernels that move take the tables with them, and with these
    the sizes of the tests on the GPU.)"""
    run("""
    for k in (b"error_tiles_dma", b"error_mid"):
        fake.fake_watch(k, 6)                                     # chunk (in columns; in blocks)
        fake.fake_watch(k, 7)                                     # slots
    def form(call):
        fake.fake_reset()
        assert call() == OK, lib.adadim_last_error(ctx)
        tiles = [c.split() for c in launched("error_") if "finish" not in c and "prologue" not in c]
        assert len(tiles) == 1, tiles
        _, name, gx, gy, block, *seen = tiles[0]
        if "error_small" in name:
            return 64, int(gx), int(gx)
        return (128, int(seen[0]), int(seen[1])) if "error_mid" in name else (256, int(seen[0]) // 256, int(seen[1]))
    ctx = context()
    for (n, out, inn), want in SCORING.items():
        arr = (c_void_p * n)(*[A.value] * n)
        shape = (c_int64(out), c_int64(inn))
        for dtype in (0, 1, 2):
            got = form(lambda: lib.adadim_layer_error_batch(ctx, n, arr, dtype, *shape, A, A, None, A))
            assert got == want, (n, out, inn, dtype, got, want)
        assert form(lambda: lib.adadim_layer_error_batch_select(ctx, n, arr, 2, *shape, A, A, None, A, A)) == want
        if n == 1:
            assert form(lambda: lib.adadim_layer_error_prepared(ctx, A, 0, *shape, A, A, None, A)) == want
    for (tokens, inn), want in GRAM.items():
        t, i = c_int64(tokens), c_int64(inn)
        for call in (lambda: lib.adadim_hessian(ctx, A, t, i, i, A, 0), lambda: lib.adadim_hessian(ctx, A, t, i, i, A, 1),
                     lambda: lib.adadim_hessian_prepared(ctx, A, t, i, i, A, A, A)):
            fake.fake_reset()
            assert call() == OK, lib.adadim_last_error(ctx)
            names = [c.split()[1] for c in launched("gram_tiles")]
            assert len(names) == 1 and ("gram_tiles_dma" in names[0]) == (want == 256), (tokens, inn, names)
    """.replace("SCORING", repr(SCORING_FORMS)).replace("GRAM", repr(GRAM_FORMS)))


def test_scoring_recording_depends_on_the_finest_cut(run):
    """Whether a scoring call can be recorded after another: when the finest cut of its contractions that is considered needs no
    more room for row partials, whatever chunk either is given."""
    run("""
    def need(n, out, inn):
        MB, NB = (out + 255) // 256, (inn + 255) // 256
        kb = NB
        while True:
            slots = sum(nb // kb + 1 for nb in range(NB))
            if kb == 1 or n * MB * slots >= 512:
                break
            kb = kb // 2 if kb > 2 else 1
        return n * (slots + 1) * out * 4
    def totals(out):
        return 8 * ((out + 255) // 256) * 8 + 256
    up = lambda n: (n + 255) // 256 * 256
    def score(ctx, n, out, inn):
        arr = (c_void_p * n)(*[A.value] * n)
        return lib.adadim_layer_error_batch(ctx, n, arr, 2, c_int64(out), c_int64(inn), A, A, None, A)
    shapes = [(1, 64, 64), (2, 512, 512), (1, 4096, 4096), (2, 1720, 2760), (2, 2048, 2048), (1, 8192, 1024), (1, 256, 11008),
              (8, 256, 4096), (3, 600, 3072), (1, 64, 16384), (2, 4096, 4096), (4, 300, 3000)]
    for a in shapes:
        for b in shapes:
            ctx = context()
            assert score(ctx, *a) == OK, lib.adadim_last_error(ctx)
            assert lib.adadim_capture_begin(ctx) == OK
            rc = score(ctx, *b)
            assert (rc == OK) == (need(*b) <= up(need(*a)) and totals(b[1]) <= up(totals(a[1]))), (a, b, rc)
            g = c_void_p()
            assert lib.adadim_capture_end(ctx, byref(g)) == OK
            lib.adadim_graph_destroy(g)
            lib.adadim_destroy(ctx)
    """)
