"""The library's host side on a stand-in for the HIP runtime (no GPU): see host_runtime.py."""
import pytest

from host_runtime import run


def test_load_after_a_refinement_that_could_not_upload(tmp_path):
    """A refinement whose topology buffer cannot be allocated (device or pinned memory) is
    refused and leaves the forest; blocks loaded and read by kernels afterwards go by that
    forest's own descriptors, never by a freed buffer."""
    run(tmp_path, '''
cfg = W.C1(jmax=6, form=W.FORM_FUSED)
lv, co = W.uniform_forest(cfg, 5)
lv, co = lv[morton(co)], co[morton(co)]
nth = 1
while True:
    s = M.Solver(cfg)
    s.init_forest(*W.uniform_forest(cfg, 1))
    s.init_forest(lv, co)
    s.load_blocks(np.zeros((len(lv), 1, cfg.npts)))
    host.host_fail_allocation(nth)
    try:
        s.refine_all()
        failed = False
    except M.MrbError as e:
        failed = True
        assert e.code == -5
    host.host_fail_allocation(0)
    if not failed:
        break
    assert s.num_blocks() == len(lv)
    data = np.random.default_rng(nth).random((len(lv), 1, cfg.npts))
    for k in range(2):
        s.load_blocks(data)
        assert host.host_scatter_faults() == 0
        pool = s.u.a.reshape(-1, cfg.npts)
        # slots of a new forest are its positions
        assert np.array_equal(pool[:len(lv)], data[:, 0]) and not pool[len(lv):].any()
    s.refine_all()
    assert s.num_blocks() == 4 * len(lv)
    s.close()
    nth += 1
assert nth > 1
''')


def test_transition_without_memory_to_remember_it(tmp_path):
    """A refinement or coarsening whose device copy for later replays cannot be allocated takes
    place all the same (kernel launched, forest changed), also where the copy would take the
    place of an older, smaller one, which is then forgotten."""
    run(tmp_path, '''
cfg = W.C1(jmax=5, form=W.FORM_FUSED)
lv, co = W.uniform_forest(cfg, 1)


def marked(s, k):
    mask = np.zeros(s.num_blocks(), np.int8)
    mask[k] = 1
    s.refine_marked(mask)
    assert host.host_null_topologies() == 0


for nth in range(1, 8):                  # every allocation of a refinement of a larger forest
    s = solver(cfg, lv, co)
    for n in range(12):                  # more transitions than are remembered
        marked(s, n % 4)
    s.init_forest(*W.uniform_forest(cfg, 3))
    s.load_blocks(np.zeros((64, 1, cfg.npts)))
    launches()
    host.host_fail_allocation(nth)
    try:
        s.refine_all()
    except M.MrbError as e:
        assert e.code == -5 and s.num_blocks() == 64 and not any("refine" in k[0] for k in launches())
    else:
        assert s.num_blocks() == 256 and any("refine" in k[0] for k in launches())
    host.host_fail_allocation(0)
    for first in range(4):               # what an entry without a copy held is planned anew
        s.init_forest(lv, co)
        s.load_blocks(np.zeros((4, 1, cfg.npts)))
        for n in range(12):
            marked(s, (first + n) % 4)
    s.close()
''')


def test_load_after_one_whose_staging_could_not_grow(tmp_path):
    """A load from host memory whose device staging cannot grow is refused; a smaller one after
    it gets a buffer of its own."""
    run(tmp_path, '''
cfg = W.C1(jmax=4, form=W.FORM_FUSED)
s = solver(cfg, *W.uniform_forest(cfg, 1))
s.init_forest(*W.uniform_forest(cfg, 3))
host.host_fail_allocation(1)
try:
    s.load_blocks(np.zeros((64, 1, cfg.npts)))
    assert False
except M.MrbError as e:
    assert e.code == -5
s.init_forest(*W.uniform_forest(cfg, 1))
data = np.random.default_rng(0).random((4, 1, cfg.npts))
s.load_blocks(data)
assert np.array_equal(s.u.a.reshape(-1, cfg.npts)[:4], data[:, 0])
''')


def test_predictor_batch_after_one_without_memory(tmp_path):
    """A batch whose workspace cannot grow (any of its buffers) is refused; a smaller one after
    it gets buffers of its own."""
    run(tmp_path, '''
cfg = W.C1(jmax=2, form=W.FORM_FUSED)
x = np.ones((64, 64), np.float32)
y, cw = np.zeros(64, np.int8), np.ones(3, np.float32)
nth = 1
while True:
    s = solver(cfg, *W.uniform_forest(cfg, 1))
    s.mlp_init(W.mlp_init_params(64, 1), np.zeros(1, np.float32), np.ones(1, np.float32))
    s.mlp_grad(x[:16], y[:16], cw)
    host.host_fail_allocation(nth)
    try:
        s.mlp_grad(x, y, cw)
        failed = False
    except M.MrbError as e:
        failed = True
        assert e.code == -5
    host.host_fail_allocation(0)
    s.mlp_grad(x[:16], y[:16], cw)
    if not failed:
        break
    nth += 1
assert nth == 13
''')


def test_launches_of_the_largest_forests(tmp_path):
    """No launch holds 2^32 threads or more, and the launches of a call have a workgroup for each
    of its work items, on 2^20 blocks of 33^2 (46 GB of pool in FP64): the tile step on whole
    blocks, 2 x 2 and 4 x 4 sub-tiles, plain and with the refinement and the analysis folded in
    (1,024 threads), the stage launches, the analysis, and the autotuner over all of them."""
    run(tmp_path, '''
cfg = W.C2(jmax=10, form=W.FORM_FUSED).replace(max_blocks=(1 << 20) + (1 << 18))
forest = {}
for l in (9, 10):
    lv, co = W.uniform_forest(cfg, l)
    order = morton(co)
    forest[l] = lv, co[order]
s = pool_free_solver(cfg, *forest[10])
s.set_topology(0)


def load(l):
    s.init_forest(*forest[l])
    s._chk(M.lib().mrb_load_blocks(s.h, 8, 1))
    launches()


def check(items, kernel, calls=1):
    got = launches()
    assert all(g * t < 2 ** 32 for _, g, t in got), got
    mine = [g for name, g, t in got if kernel in name]
    assert sum(mine) >= calls * items and len(mine) >= calls, (kernel, items, got)


n = 1 << 20
s.set_sweep(3)
for nsub, tpb in ((1, 1024), (2, 1024), (4, 256)):
    s.tune(nsub=nsub, reps=-tpb)
    load(10)
    s.rk4(0.0, cfg.dt)
    check(n * nsub * nsub, "k_rk4t")
    load(9)
    s.step(0.0, cfg.dt)                      # level 9 refined to level 10 inside the tile launch
    check(n * nsub * nsub, "k_rk4t")
load(10)
s.set_sweep(0)
s.tune()
s.rk4(0.0, cfg.dt)
check(n, "k_stage", 4)
s.mr_pass()
check(n, "k_mr")
s.set_sweep(2)
s.tune(reps=1)
check(n, "k_rk4t")
''')


@pytest.mark.parametrize("units,level,last", [(32, 2, 5), (256, 4, 0)])
def test_navier_stokes_split_goes_by_the_devices_compute_units(tmp_path, units, level, last):
    """The Navier-Stokes stage and filter take halves of blocks up to a block per compute unit of
    the device at hand and thirds beyond, in both precisions: uniform forests with `last` or
    more of their blocks refined, 31 and 34 blocks on 32 units, 256 and 259 on 256."""
    run(tmp_path, f'''
host.host_compute_units({units})
for precision in (W.FP64, W.MIXED):
    cfg = W.DSL(jmax=6, form=W.FORM_FUSED, precision=precision).replace(max_blocks=2000)
    for refined, parts in (({last}, 2), ({last} + 1, 3)):
        lv, co = W.uniform_forest(cfg, {level})
        kids = np.concatenate([2 * co[:refined] + np.array([i, j]) for i in (0, 1) for j in (0, 1)])
        lv = np.r_[lv[refined:], np.full(len(kids), {level} + 1, np.int8)]
        co = np.r_[co[refined:], kids.astype(np.int32)]
        s = pool_free_solver(cfg, lv, co)
        s.rk4(0.0, cfg.dt)
        got = [(name, g) for name, g, t in launches()]
        want = (parts * len(lv) + 7) // 8 * 8
        assert [g for name, g in got if "k_stage_ns" in name] == [want] * 4, (len(lv), got)
        assert [g for name, g in got if "k_filter2" in name] == [want], (len(lv), got)
        s.close()
''')


def test_stats_name_the_workgroups_that_run(tmp_path):
    """stage_threads and stage_parts are those of a launch over the current grid, stage_ran those
    of the last launch, analysis_workgroup the analysis's; every shape, precision and split."""
    run(tmp_path, '''
for make, level in ((W.C1, 3), (W.C2, 2), (W.C2, 3), (W.DSL, 3), (W.DSL, 4), (W.DSL, 5), (W.C4, 2)):
    for precision in (W.FP64, W.MIXED):
        cfg = make(jmax=6, form=W.FORM_FUSED, precision=precision).replace(max_blocks=6000)
        lv, co = W.uniform_forest(cfg, level)
        s = pool_free_solver(cfg, lv, co)
        for nsub, reps in ((0, 0), (2, 0), (0, 1)):
            s.tune(nsub=nsub, reps=reps)
            if reps:
                keys = s.stats()["tune_ms"]
                ran = {(g, t) for name, g, t in launches() if "k_stage" in name}
                for k in keys:
                    if k.startswith("1t") and not k.endswith("L"):
                        t, p = (k[2:].split("p") + ["1"])[:2]
                        assert ((len(lv) * int(p) + 7) // 8 * 8, int(t)) in ran, (k, ran)
            launches()
            s.set_sweep(0)
            s.rk4(0.0, cfg.dt)
            s.mr_pass()
            st = s.stats()
            got = launches()
            stage = {(g, t) for name, g, t in got if "k_stage" in name}
            (wg, t), = stage
            assert st["stage_threads"] == t and st["stage_ran"] == [st["stage_parts"], t], (cfg.name, st, got)
            items = (len(lv) * st["stage_parts"] + 7) // 8 * 8
            assert wg == (min(items, st["grid"]) if t == 256 else items)   # (256: a loop over items)
            (t,) = {t for name, g, t in got if "k_mr" in name}
            assert st["analysis_workgroup"] == t, (cfg.name, st, got)
            # a larger grid: the last launch keeps its name
            s.refine_all()
            assert s.stats()["stage_ran"] == st["stage_ran"]
            s.init_forest(lv, co)
            s._chk(M.lib().mrb_load_blocks(s.h, 8, 1))
            launches()
        s.close()
''')


def test_whole_blocks_can_be_forced_for_every_shape(tmp_path):
    """tune(nsub=1) is accepted for every shape and precision and takes the kernel that the
    default and the autotuner mean by one sub-tile; workgroup sizes are named by reps < 0 as
    before, and what is not compiled is refused as before."""
    run(tmp_path, '''
for make, level, zone, points in ((W.C1, 3, "k_stage2", 256), (W.C2, 3, "k_stage2", 512), (W.DSL, 3, "k_stage_ns", 1024),
                                  (W.C4, 2, "k_stage3", 512)):
    for precision in (W.FP64, W.MIXED):
        cfg = make(jmax=6, form=W.FORM_FUSED, precision=precision).replace(max_blocks=6000)
        s = pool_free_solver(cfg, *W.uniform_forest(cfg, level))
        s.set_sweep(0)

        def stage():
            launches()
            s.rk4(0.0, cfg.dt)
            return " ".join(sorted({name for name, g, t in launches() if "k_stage" in name}))

        default = stage()
        assert zone in default
        for reps in (0, -{"k_stage2": 448 if cfg.bs == 17 else 384, "k_stage_ns": 576, "k_stage3": 448}[zone]):
            s.tune(nsub=2)
            assert "7k_stage" in stage()
            assert s.tune(nsub=1, reps=reps) == 1
            assert stage() == default, (cfg.name, precision)
            assert s.stats()["stage_tiles"] == 1
        chosen = s.tune(reps=1)
        assert s.tune(nsub=chosen) == chosen
        try:                                   # the point-owner kernel, where it is compiled
            s.tune(nsub=1, reps=-points)
            assert (zone if (cfg.name, precision) == ("DSL", W.FP64) else "7k_stage") in stage()
        except M.MrbError as e:
            assert e.code == -1 and (cfg.name, precision) == ("C4", W.FP64)
        for bad in ((3, 0), (1, -768), (8, 0)):
            try:
                s.tune(nsub=bad[0], reps=bad[1])
                assert False, bad
            except M.MrbError as e:
                assert e.code == -1
        s.close()
''')


@pytest.mark.parametrize("units", [64, 256])
def test_default_stage_of_few_blocks(tmp_path, units):
    """Blocks of 33^2 take 4 x 4 sub-tiles while these are fewer than two workgroups a compute
    unit (advection) or at most one (Navier-Stokes), whole blocks beyond."""
    run(tmp_path, f'''
units = {units}
host.host_compute_units(units)
for make, last in ((W.C2, units // 8 - 1), (W.DSL, units // 16)):
    for precision in (W.FP64, W.MIXED):
        cfg = make(jmax=4, form=W.FORM_FUSED, precision=precision).replace(max_blocks=500)
        seen = set()
        for refined in range(13):
            for level in (1, 2):
                lv, co = W.uniform_forest(cfg, level)
                if refined > len(lv):
                    continue
                kids = np.concatenate([2 * co[:refined] + np.array([i, j]) for i in (0, 1) for j in (0, 1)])
                lv = np.r_[lv[refined:], np.full(len(kids), level + 1, np.int8)]
                co = np.r_[co[refined:], kids.astype(np.int32)]
                s = pool_free_solver(cfg, lv, co)
                s.rk4(0.0, cfg.dt)
                tiled = any("7k_stage" in name for name, g, t in launches())
                assert tiled == (len(lv) <= last), (cfg.name, len(lv), last)
                assert s.stats()["stage_tiles"] == (4 if tiled else 1)
                seen.add(tiled)
                s.close()
        assert seen == {{True, False}}
''')


def test_default_stage_of_many_small_blocks(tmp_path):
    """Forests of 49,152 blocks of 17^2 and more take the point-owner kernel on whole blocks,
    smaller ones and other shapes of as many blocks the zone-owner kernel; forcing whole blocks
    still means the latter."""
    run(tmp_path, '''
def refined(cfg, level, k):
    lv, co = W.uniform_forest(cfg, level)
    order = morton(co)
    lv, co = lv[order], co[order]
    kids = np.concatenate([2 * co[:k] + np.array([i, j]) for i in (0, 1) for j in (0, 1)])
    return np.r_[lv[k:], np.full(len(kids), level + 1, np.int8)], np.r_[co[k:], kids.astype(np.int32)]


for precision in (W.FP64, W.MIXED):
    for make, k, want in ((W.C1, 10922, "k_stage2"), (W.C1, 10923, "7k_stage"), (W.C2, 10923, "k_stage2")):
        cfg = make(jmax=8, form=W.FORM_FUSED, precision=precision).replace(max_blocks=50000)
        lv, co = refined(cfg, 7, k)
        s = pool_free_solver(cfg, lv, co)
        s.rk4(0.0, cfg.dt)
        got = [(name, t) for name, g, t in launches() if "k_stage" in name]
        assert len(got) == 4 and all(want in name for name, t in got), (cfg.name, len(lv), got)
        assert s.stats()["stage_threads"] == got[0][1] and s.stats()["stage_tiles"] == 1
        s.tune(nsub=1)
        s.rk4(0.0, cfg.dt)
        assert all("k_stage2" in name for name, g, t in launches())
        s.close()
''')
