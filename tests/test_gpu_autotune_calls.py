"""The sweep autotuner times what a call runs: on a band whose buffers exceed the
Infinity Cache every candidate's time is that of its sweeps in a call of many,
the first one the default's.  Timings of one card differ by a few percent; sweeps
that all read one buffer were up to 40 % off.  phi is only read, and the picked
configuration gives the bits of the default."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_autotuned_times_are_those_of_calls():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_11473_amd as sg
    from paper_2512_11473_amd import workload
    cfg = synth.config_shell()
    wl = workload.setup(cfg["shape"], cfg["N"], cfg["noise_amp"], cfg["noise_seed"])
    g = wl.grid
    assert 2 * g.n_total * 256 > 1 << 28
    wl.reset()
    start = wl.phi.clone()

    def call(n_iter):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        wl.phi.copy_(start)
        a.record()
        sg.reinitialize(g, wl.phi, wl.scratch, n_iter)
        b.record()
        torch.cuda.synchronize()
        return 1e3 * a.elapsed_time(b) / n_iter

    try:
        sg.set_sweep_config(0, 1)
        call(5)
        want = wl.phi.clone()
        wl.phi.copy_(start)
        v, groups, table = sg.autotune_sweep(g, wl.phi, wl.scratch, reps=20)
        assert torch.equal(wl.phi, start)
        call(5)
        assert torch.equal(wl.phi, want)
        assert (v, groups) == sg.SWEEP_TUNE_CANDIDATES[int(table.argmin())]
        table = np.minimum(table, sg.autotune_sweep(g, wl.phi, wl.scratch, reps=20)[2])   # the calls' are the least of three
        for c, us in zip(sg.SWEEP_TUNE_CANDIDATES, table):
            sg.set_sweep_config(*c)
            in_call = min(call(40) for _ in range(3))
            print(c, us, in_call, flush=True)
            assert 0.8 < us / in_call < 1.25, (c, us, in_call)
    finally:
        sg.set_sweep_config(0, 1)
    g.destroy()
