"""GPU checks that tuning does not choose what is slower than no tuning, and that
schedules timed on older kernels are not taken from a cache."""
import json

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def test_no_schedule_is_a_candidate(tmp_path):
    """14 sites in FP64, where the automatic choice takes a kernel that no schedule asks
    for: it is timed as well, and the choice is the fastest up to two ties of 1 %."""
    from paper_0706_3293_amd import autotune, inputs
    J = inputs.ring_couplings(14, -1.0, -0.3)
    cache = str(tmp_path / "tune.json")
    b, sched = autotune.tuned_basis(14, J, dtype=torch.float64, reps=20, cache=cache)
    (entry,) = json.load(open(cache)).values()
    timed = {tuple(s): ms for s, ms in entry["trials"]}
    print(sched, entry["ms"], timed[(0, 0, 0, 0, 0)], min(timed.values()), flush=True)
    assert (0, 0, 0, 0, 0) in timed
    assert entry["ms"] <= 1.021 * min(timed.values())
    assert autotune.tune(14, J, dtype=torch.float64, cache=cache) == sched
    v = torch.tensor(inputs.start_vector(b.dim, 0), device="cuda")
    assert b.lanczos(J, v, 10).steps_done == 10


def test_schedules_of_older_kernels_are_tuned_again(tmp_path):
    import hashlib

    import numpy as np

    from paper_0706_3293_amd import Basis, autotune, inputs
    cache = str(tmp_path / "tune.json")
    J = inputs.ring_couplings(12, -1.0, -0.3)
    h = hashlib.sha1(np.ascontiguousarray(J).tobytes()).hexdigest()[:16]
    shapes = hashlib.sha1(b"12/1/0;12/1/0").hexdigest()[:16]
    old = {f"passA:N=12,2M=0,dtype={torch.float64},J={h}": {"schedule": [8, 64, 8, 1, 64]},
           f"batched:n=2,nvec=2,steps=6,shapes={shapes}": {"schedule": [63, 7]}}
    json.dump(old, open(cache, "w"))
    assert autotune.tune(12, J, dtype=torch.float64, reps=2, cache=cache) != (8, 64, 8, 1, 64)
    bases = [Basis(12, two_s=1, two_M=0) for _ in range(2)]
    V0s = [np.ones((2, b.dim)) + np.arange(b.dim) / b.dim for b in bases]
    best = autotune.tune_batched(bases, [J, J], V0s, 6, reps=1, cache=cache)
    assert best != (63, 7) and best in autotune.BATCH_CANDIDATES
    assert set(old) < set(json.load(open(cache)))
