"""Host code of plans, schedules and launch shapes on the CPU, with a stand-in for the HIP runtime (no
kernel runs): calls that must not end the process, and launches that must stay within a grid's limits."""

import pytest

from tests import hip_stub


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("hip_stub")
    return lambda script: hip_stub.run(tmp, script)


@pytest.mark.parametrize("kw", ["[(65536, 65536)]", "[(480, 640)], in_pitches=[1 << 24]",
                                "[(480, 640)], out_pitches=[1 << 29]", "[(480, 640), (65536, 65536), (480, 640)]"])
def test_schedule_of_planes_beyond_the_strip_kernel(host, kw):
    """The schedule of a plan with a plane of 4 GiB or more (or 16 output rows of as much)."""
    sched = host(f"""
f = aol.Polyphase(3, 8, synthgen.design_taps(3, 8, 11))
plan = aol.DownscalePlan({kw}, hf=f, vf=f)
print(json.dumps([plan.schedule(1), plan.schedule(300)]))
""")
    for s, n in zip(sched, (1, 300)):
        assert s["kernel"] == "band" and s["items"] == n * s["units_per_frame"] > 0, s


def test_batch_segments_of_any_length(host):
    """The longest segment a caller may name, on streams of many 16-row blocks."""
    sched = host("""
f = aol.Polyphase(16, 24, synthgen.design_taps(16, 24, 9))
plan = aol.BatchPlan([(1080, 1920, f, f), (1080, 1921, f, f)])
plan.set_schedule(2 ** 31 - 16, 150 * 1024)
long = json.loads(plan.schedule())
plan.set_schedule(1024, 150 * 1024)
print(json.dumps([long, json.loads(plan.schedule())]))
""")
    assert sched[0]["seg"] == 2 ** 31 - 16 and sched[0]["units"] == sched[1]["units"] > 0


def test_batch_output_of_2_32_rows(host):
    """A stream whose output height is 2^32 (zero in 32 bits) makes a plan or is refused."""
    units = host("""
v, h = aol.Polyphase(16, 1, [[256]] * 16), aol.Polyphase(1, 1, [[256]])
try:
    print(json.dumps(json.loads(aol.BatchPlan([(1 << 28, 1, h, v)]).schedule())["units"]))
except aol.AolError as e:
    print(json.dumps(e.status))
""")
    assert units > 0 or units == -2


LINEAR = """
def kernel(shape, rep, pat, origin, paving, fitting, oshape, opaving, ofitting, opat, value=1):
    n_in, n_out = int(np.prod(pat)), int(np.prod(opat))
    tin = aol.make_tiler(shape, rep, pat, origin, paving, fitting)
    tout = aol.make_tiler(oshape, rep, opat, (0,) * len(oshape), opaving, ofitting)
    plan = aol.aol_linear_plan_create(tin, tout, np.full((n_out, n_in), value))
    stub.stub_reset()
    aol.aol_linear_run(plan, BUF, 2 * BUF, 0)
    aol.aol_linear_plan_destroy(plan)
    return launches()[0][0]
"""


def test_linear_packed_form_strides(host):
    """Pavings of -2^63 (a residue of any modulus, but no stride that fits 64 bits) stay off the packed form."""
    names = host(LINEAR + """
def rgb(p):
    return kernel((30000,), (3, 500), (3,), (0,), [[p, 3]], [[1]], (3, 3, 500), [[0, 0], [1, 0], [0, 1]], [[1], [0], [0]], (3,))
print(json.dumps([rgb(1500), rgb(-2 ** 63)]))
""")
    assert "k_linear_pack" in names[0] and "k_linear_pack" not in names[1], names


def test_linear_matrix_core_form_axes(host):
    """Axes above 2^30 stay off the matrix-core form, whose coordinates are sums of two in 32 bits."""
    names = host(LINEAR + """
def fir(n):
    return kernel((n,), (16, 400), (64,), (n - 5,), [[0, 1]], [[1]], (16, 400, 8), [[1, 0], [0, 1], [0, 0]], [[0], [0], [1]], (8,))
print(json.dumps([fir(2 ** 30), fir(2 ** 30 + 1), fir(2 ** 31 - 1)]))
""")
    assert "k_linear_box" in names[0], names
    assert all("k_linear_box" not in n for n in names[1:]), names


@pytest.mark.parametrize("rep,paving", [((8192, 8192, 4), [[1, 0, 9], [0, 1, 3], [0, 0, 1]]),
                                        ((2 ** 24 + 9, 2, 1), [[1, 0, 0], [3, 0, 0], [0, 1, 0]])])
def test_weighted_sum_grids(host, rep, paving):
    """Repetition spaces of more blocks than a grid holds (2^32 threads): cut into several launches that
    together hold every block, plan and one-shot form."""
    counts = host(f"""
rep, paving = {rep}, {paving}
tin = aol.make_tiler((64, 70, 70), rep, (9,), (0, 0, 0), paving, [[1], [0], [0]])
plan = aol.aol_wsum_plan_create(tin, aol.identity_out_tiler(rep), np.ones(9))
n = []
for run in (lambda: aol.aol_wsum_run(plan, BUF, 2 * BUF, 0),
            lambda: aol.aol_weighted_sum_f32(tin, aol.identity_out_tiler(rep), np.ones(9), BUF, 2 * BUF, 0)):
    stub.stub_reset()
    run()
    assert all(g * b < 2 ** 32 for _, g, b in launches())
    n.append(sum(g for _, g, _ in launches()))
print(json.dumps(n))
""")
    points = rep[0] * rep[1] * rep[2]
    assert counts[0] == counts[1] >= points // (64 * 64), counts


def test_weighted_sum_short_lane_dimension(host):
    """The direct form's threads nearly all have a point, however short the dimension of its lanes."""
    got = host("""
got = []
for lane in (2, 3, 4, 8, 16, 32, 64):
    rep = (1 << 18, lane)
    tin = aol.make_tiler(((1 << 18) + 70, lane), rep, (9,), (0, 0), [[1, 7], [0, 1]], [[1], [0]])
    plan = aol.aol_wsum_plan_create(tin, aol.identity_out_tiler(rep), np.ones(9))
    stub.stub_reset()
    aol.aol_wsum_run(plan, BUF, 2 * BUF, 0)
    got.append([launches()[0][0], sum(g * b for _, g, b in launches()) / (rep[0] * rep[1])])
print(json.dumps(got))
""")
    for name, threads_per_point in got:
        assert "k_wsumILb0E" in name and threads_per_point <= 1.4, got


def test_linear_matrix_core_form_only_where_it_pays(host):
    """Dense windows run on the matrix cores; patterns with few elements in a 16-byte chunk and few
    outputs point by point (as products 2.1 to 2.5 times slower)."""
    names = host(LINEAR + """
def window(n, k, d, n_out, value, q=1):
    return kernel((n * q, n * q), (n, n), k, (0, 0), [[q, 0], [0, q]], [[d[0], 0], [0, d[1]]],
                  (n, n, n_out), [[1, 0], [0, 1], [0, 0]], [[0], [0], [1]], (n_out,), value)
print(json.dumps([[window(300, (17, 17), (1, 1), 9, 1, 8), window(1000, (12, 12), (1, 1), 1, 1), window(60, (8, 8), (1, 1), 4, 300)],
                  [window(1000, (33, 1), (1, 1), 1, 1), window(1000, (1, 33), (3, 20), 2, 300), window(1000, (7, 7), (3, 20), 1, 300),
                   window(60, (8, 8), (1, 1), 1, 1, 16)]]))
""")
    assert all("k_linear_box" in n for n in names[0]), names
    assert all("k_linear_box" not in n for n in names[1]), names


TUNE = """
stub.stub_elapsed.argtypes = [ctypes.POINTER(ctypes.c_float), ctypes.c_int]
f = aol.Polyphase(3, 8, synthgen.design_taps(3, 8, 11))
def tuned(cache, times):
    plan = aol.BatchPlan([(480, 640, f, f)] * 5, tune_cache=cache)
    aol.aol_batch_set_pointers(plan._h, aol._ptrs([BUF] * 5), aol._ptrs([BUF] * 5), 0)
    stub.stub_elapsed((ctypes.c_float * len(times))(*times), len(times))
    aol.aol_autotune(plan._h, 0)
    return json.loads(plan.schedule())
"""


def test_autotune_times_the_default(host, tmp_path):
    """A tuned batch is no slower than an untuned one: the default schedule is among the candidates (here
    the first one timed is the fastest)."""
    sched, again = host(TUNE + f"""
cache = {str(tmp_path / "tune.txt")!r}
sched = tuned(cache, [0.5] * 3)
print(json.dumps([sched, json.loads(aol.BatchPlan([(480, 640, f, f)] * 5, tune_cache=cache).schedule())]))
""")
    assert sched["seg"] == 0 and not any(sched["class_segs"]) and again == sched, (sched, again)


def test_tuning_cache_names_the_kernel(host, tmp_path):
    """A line tuned for the column-band kernel (the plain key) is not applied to the strip kernel, nor the
    other way round (a batch with a stream beyond the strip kernel runs the column-band kernel)."""
    got = host(TUNE + f"""
cache = {str(tmp_path / "tune.txt")!r}
tuned(cache, [0.5] * 6 + [0.1] * 3)
key = open(cache).read().split()[0]
plain = key[:-len("|strip")] if key.endswith("|strip") else key
seg = lambda shapes, **kw: json.loads(aol.BatchPlan([(h, w, f, f, ip, 0) for h, w, ip in shapes], **kw).schedule())["seg"]
got = [seg([(480, 640, 640)] * 5, tune_cache=cache)]
open(cache, "w").write(plain + " 128 153600 0 1000\\n")
got += [seg([(480, 640, 640)] * 5, tune_cache=cache), seg([(480, 640, 1 << 24)] * 5, tune_cache=cache)]
open(cache, "w").write(plain + "|strip 64 153600 0 1000\\n")
got += [seg([(480, 640, 640)] * 5, tune_cache=cache), seg([(480, 640, 1 << 24)] * 5, tune_cache=cache)]
print(json.dumps(got))
""")
    assert got == [32, 0, 128, 64, 0], got


def test_plan_uploads_what_its_kernel_reads(host):
    """A plan on the strip kernel uploads no unit lists of the column-band kernel (at creation and when a
    schedule is named); a plan beyond the strip kernel does."""
    got = host("""
f = aol.Polyphase(3, 8, synthgen.design_taps(3, 8, 11))
got = []
for pitches in (None, [1 << 24]):
    stub.stub_reset()
    plan = aol.DownscalePlan([(1080, 1920)], f, f, in_pitches=pitches)
    got.append(stub.stub_copies())
    stub.stub_reset()
    plan.set_band(0, 32)
    got.append(stub.stub_copies())
print(json.dumps(got))
""")
    assert got[2] - got[0] >= 8 and got[3] - got[1] >= 6, got


def test_schedule_reports_the_launch(host):
    """The "runs" part of a plan's schedule is the launch that is made."""
    got = host("""
f = aol.Polyphase(3, 8, synthgen.design_taps(3, 8, 11))
got = []
for shapes, kw in (([(1080, 1920), (540, 960), (540, 960)], {}), ([(768, 1366)], {}), ([(480, 640)], dict(precision="bf16")),
                   ([(480, 640)], dict(in_pitches=[1 << 24])), ([(480, 640)], dict(seg=32))):
    seg = kw.pop("seg", 0)
    plan = aol.DownscalePlan(shapes, f, f, **kw)
    if seg:
        plan.set_band(0, seg)
    for n in (1, 3, 40, 300):
        stub.stub_reset()
        fn = aol.aol_downscale_f if kw.get("precision") else aol.aol_downscale_u8
        k = len(shapes)
        fn(plan._h, n, [BUF] * k, [1 << 34] * k, [BUF] * k, [1 << 34] * k, 0)
        got.append([plan.schedule(n)["runs"], launches()])
print(json.dumps(got))
""")
    for runs, made in got:
        assert len(made) == 1, made
        name, grid, block = made[0]
        assert f"k_{runs['kernel']}I" in name and runs["workgroups"] == grid and runs["waves"] * 64 == block, (runs, made)
    assert {r["kernel"] for r, _ in got} == {"strip", "band"} and {r["waves"] for r, _ in got} == {4, 8, 16}
