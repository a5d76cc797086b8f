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
