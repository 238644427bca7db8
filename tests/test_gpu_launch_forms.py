"""GPU: the launches and allocations a run makes, counted in a process of its own (hip_calls)."""

import pytest

import hip_calls

pytestmark = pytest.mark.gpu


REFUSED = r"""
out = []
c = Case(np.random.default_rng(1300), 240, 250, 16, 9, noise=0.05)
for refuse in (0, 240 * 250 * 8, 64 * 16 * 16 * 8):   # none; the object's second buffer; the staging's
    g = c.gpu(3, 0.5)
    g.run_minibatch(np.arange(64, dtype=np.int32))    # the plain staging is there
    calls.refuse(refuse)
    calls.start()
    g.run_epochs(2, 64, seed=7)
    launches = calls.stop().count('k')
    calls.refuse(0)
    out.append([launches, g.get_object().view(np.uint32).tolist()])
    g.run_epochs(1, 64, seed=9)
    out[-1].append(g.get_object().view(np.uint32).tolist())
    g.close()
n = (c.n_pos + 63) // 64
print(json.dumps([n, [o[0] for o in out], [o[1:] == out[0][1:] for o in out]]))
"""


def test_run_without_the_merged_launches_buffers(tmp_path):
    """Where the second buffers of merged launches cannot be allocated the epochs run as two
    launches per minibatch, to the same object."""
    n, launches, equal = hip_calls.run(tmp_path, REFUSED)
    assert launches == [2 * n + 2, 4 * n, 4 * n]   # two chunks of one epoch
    assert equal == [True, True, True]


AUTOTUNE = r"""
c = Case(np.random.default_rng(1301), 240, 250, 16, 9, noise=0.05)
g = c.gpu(3, 0.5)
calls.start()
g.autotune_batch([8, 16, 64, 32, 128], 1)
print(json.dumps(calls.stop()))
"""


def test_batch_autotuner_allocates_before_its_trials(tmp_path):
    """Every allocation of magpie_autotune_batch precedes its first launch, so none falls into a
    candidate's timing."""
    trace = hip_calls.run(tmp_path, AUTOTUNE)
    assert "k" in trace and "m" in trace
    assert "m" not in trace[trace.index("k"):]
