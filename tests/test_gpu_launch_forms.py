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


# m, rows, cols, step, levels, batch, epochs: on both sides of the rules' lines
FORMS = [
    (16, 90, 131, 9, 3, 8, 10, "chained"),
    (16, 90, 131, 9, 3, 9, 2, "merged"),
    (16, 240, 250, 9, 5, 256, 10, "merged"),
    (16, 100, 110, 3, 2, 128, 1, "two"),        # 12 windows of a minibatch overlap another
    (32, 128, 128, 12, 2, 4, 10, "chained"),
    (32, 128, 128, 12, 2, 8, 3, "merged"),
    (32, 128, 128, 12, 2, 16, 3, "two"),
    (32, 128, 128, 12, 6, 1, 2, "chained"),     # V-cycle through LDS
    (32, 128, 128, 12, 6, 2, 2, "merged"),
    (32, 500, 490, 17, 6, 128, 2, "merged"),    # the largest minibatch of its plan
    (32, 500, 490, 17, 3, 100, 10, "merged"),
    (32, 403, 390, 17, 6, 128, 2, "two"),
    (64, 180, 190, 16, 3, 1, 2, "chained"),
    (64, 180, 190, 16, 3, 2, 2, "two"),
]

EQUAL = r"""
out = []
for m, rows, cols, step, levels, batch, epochs, form in arg:
    c = Case(np.random.default_rng(1303 + m + batch), rows, cols, m, step, noise=0.05)
    c.offs[0] = c.offs[1]                        # one position measured twice
    c.offs[-1] = (rows - m, cols - m)            # a window in the corner
    got = []
    for timing in (False, True):
        g = c.gpu(levels, 0.5)
        g.set_timing(timing)
        calls.start()
        g.run_epochs(epochs, batch, seed=7)
        trace = calls.stop()
        got.append((g.get_object().view(np.uint32), g.step_phi(), trace.count('k'), trace.count('t')))
        g.close()
    (za, pa, ka, ta), (zb, pb, kb, tb) = got
    out.append([(c.n_pos + batch - 1) // batch, ka, ta, tb, bool(np.array_equal(za, zb) and np.array_equal(pa, pb))])
print(json.dumps(out))
"""


def test_launch_forms_and_their_results(tmp_path):
    """Each case takes the form named, by its number of launches, and gives the objects and per-position
    objectives of timed epochs (two launches per minibatch) bit for bit."""
    for case, (n, untimed, stray, timed, equal) in zip(FORMS, hip_calls.run(tmp_path, EQUAL, FORMS)):
        epochs, form = case[6], case[7]
        chunks = 1 + -(-(epochs - 1) // 8)       # of 1, 8, 8, ... epochs
        want = {"chained": chunks, "merged": n * epochs + chunks, "two": 2 * n * epochs}[form]
        print(case, n, untimed, timed, flush=True)
        assert timed == 2 * n * epochs and stray == 0, case
        assert untimed == want, case
        assert equal, case


LONG = r"""
c = Case(np.random.default_rng(1304), 60, 66, 16, 7, noise=0.05)
got = []
for form in ("noalloc", "epochs", "timed"):
    g = c.gpu(3, 0.5)
    g.set_timing(form == "timed")
    calls.start()
    (g.run_epochs_noalloc if form == "noalloc" else g.run_epochs)(200, 1, seed=7)
    trace = calls.stop()
    got.append((g.get_object().view(np.uint32), trace.count('k')))
    g.close()
big = Case(np.random.default_rng(1305), 230, 236, 16, 3, noise=0.05)
for timing in (False, True):
    g = big.gpu(3, 0.5)
    g.set_timing(timing)
    calls.start()
    g.run_epochs(1, 1, seed=7)
    trace = calls.stop()
    got.append((g.get_object().view(np.uint32), trace.count('k')))
    g.close()
same = [bool(np.array_equal(got[i][0], got[2][0])) for i in range(2)] + [bool(np.array_equal(got[3][0], got[4][0]))]
print(json.dumps([c.n_pos, got[0][1], got[1][1], big.n_pos, got[3][1], same]))
"""


def test_long_chains_are_cut(tmp_path):
    """A chained launch takes at most 4096 minibatches, in the middle of an epoch too."""
    n, noalloc, epochs, big, one_epoch, same = hip_calls.run(tmp_path, LONG)
    assert 200 * n > 4096 and 4096 % n and big > 4096
    assert noalloc == 1 + -(-200 * n // 4096)        # the permutations of one chunk, then the chain
    assert epochs == 26                              # 1 epoch, then 24 chunks of 8 and one of 7
    assert one_epoch == -(-big // 4096)
    assert same == [True, True, True]
