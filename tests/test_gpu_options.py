"""Launch fields of chem_opts: each changes what it stands for and nothing else,
so the ones that only schedule leave every bit of a default call as it is."""
import numpy as np
import pytest

from paper_2506_02602_amd import workloads as wl

from gpu_common import to_gpu

pytestmark = pytest.mark.gpu

FIELDS = [dict(block_size=64), dict(block_size=128), dict(block_size=512), dict(chunk_steps=1),
          dict(chunk_steps=8), dict(pool_order=-1), dict(pool_order=1), dict(pool_order=3),
          dict(block_size=192, chunk_steps=4, pool_order=2)]


@pytest.mark.parametrize("n", [2000, 30000])
@pytest.mark.parametrize("entry", ["integrate", "noalloc", "batched", "graph"])
def test_scheduling_fields_keep_the_bits(mech9_path, n, entry):
    """A small pool (the cooperative kernel alone) and one with a tail list."""
    import torch
    from paper_2506_02602_amd import chemgpu as cg
    s0, hot = wl.front_2d(mech9_path, nx=1024, ny=1024, seed=93)
    k = n // 2
    s = np.ascontiguousarray(np.concatenate([s0[:, hot][:, :k], s0[:, ~hot][:, :n - k]], axis=1))
    gm = cg.chem_mech_load(mech9_path)
    cg.chem_workspace_reserve(gm, n)

    def run(**kw):
        o = cg.make_opts(**kw)
        st = to_gpu(s)
        counts = torch.zeros(2 * n, dtype=torch.int32, device="cuda")
        box = [dict(state=st, dt=wl.DT_FLOW, n_sub=1, counts=counts)]
        if entry == "integrate":
            cg.chem_integrate(gm, st, wl.DT_FLOW, o, counts=counts)
        elif entry == "noalloc":
            cg.chem_integrate_noalloc(gm, st, wl.DT_FLOW, o, counts=counts)
        elif entry == "batched":
            cg.chem_integrate_batched(gm, box, o)
        else:
            g = cg.chem_graph_capture_batched(gm, box, o)
            g.launch()
            torch.cuda.synchronize()
            g.close()
        torch.cuda.synchronize()
        return st, counts
    ref = run()
    assert int(ref[1].max()) > 40      # past every hand-off point
    for kw in FIELDS:
        got = run(**kw)
        assert torch.equal(ref[0], got[0]) and torch.equal(ref[1], got[1]), kw
    gm.close()


@pytest.mark.parametrize("n", [64, 3000])
def test_tuning_keeps_the_direct_launch(mech9_path, n):
    """The autotuner times the launch of a call that names nothing: for a pool that
    the cooperative kernel takes as it is (where everything else first steps the
    cells one per lane, three times as long) that launch stays, for tuned calls
    and with the options it returns, bit for bit; a larger pool of the same size
    bucket does not change it."""
    import torch
    from paper_2506_02602_amd import chemgpu as cg
    s0, hot = wl.front_2d(mech9_path, nx=1024, ny=1024, seed=94)
    s = np.ascontiguousarray(s0[:, hot][:, :n])
    gm = cg.chem_mech_load(mech9_path)
    cg.chem_workspace_reserve(gm, 8000)

    def run(opts=None):
        st = to_gpu(s)
        cg.chem_set_kernel_timing(gm, True)
        cg.chem_integrate(gm, st, wl.DT_FLOW, opts)
        torch.cuda.synchronize()
        kt = cg.chem_kernel_times(gm)
        cg.chem_set_kernel_timing(gm, False)
        return st, kt["coop"] > 10 * kt["persistent"]
    ref, direct = run()
    assert direct
    best = cg.chem_autotune(gm, [dict(state=to_gpu(s), dt=wl.DT_FLOW)], reps=1)
    for opts in (None, best):
        got, direct = run(opts)
        assert direct and torch.equal(got, ref)
    if n > 2048:
        big = np.ascontiguousarray(s0[:, hot][:, :8000])
        cg.chem_autotune(gm, [dict(state=to_gpu(big), dt=wl.DT_FLOW)], reps=1)
        s = np.ascontiguousarray(s0[:, hot][:, :4500])     # 4,097 to 8,192: the same bucket
        assert run()[1]
    gm.close()


@pytest.mark.parametrize("opt", [{}, dict(tail_steps=-1), dict(scheme="rkf45")])
def test_tiny_absolute_tolerance(mech9_path, opt):
    """An absolute tolerance below the smallest normal number: cells of an inert
    gas, whose errors are all zero, still take their one step."""
    import torch
    from paper_2506_02602_amd import chemgpu as cg
    names, W = wl.read_species(mech9_path)
    n = 100
    Y = np.zeros((len(names), n))
    Y[names.index("N2")] = 1.0
    T = np.linspace(400.0, 2500.0, n)
    s = wl.pack(T, Y, wl.density(T, np.full(n, wl.P_ATM), Y, W))
    gm = cg.chem_mech_load(mech9_path)
    cg.chem_workspace_reserve(gm, n)
    st, status = to_gpu(s), torch.full((n,), -1, dtype=torch.int32, device="cuda")
    cg.chem_integrate(gm, st, wl.DT_FLOW, cg.make_opts(atol=1e-310, **opt), status=status)
    torch.cuda.synchronize()
    assert (status == 0).all()
    assert np.array_equal(st.cpu().numpy()[:10], s[:10])
    gm.close()
