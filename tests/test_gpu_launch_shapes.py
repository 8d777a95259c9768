"""Launch shapes chosen by a call's size, at the sizes where one gives way to
the next, against the CPU oracle.  Integer work: tolerance 0."""
import numpy as np
import pytest

import oracle
from paper_2603_10242_amd import workload as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ace(need_gpu):
    import torch
    from paper_2603_10242_amd import ace as A
    A.load()
    torch.cuda.set_device(0)
    A.set_tuning(**A.default_tuning())
    yield A
    A.set_tuning(**A.default_tuning())


@pytest.mark.parametrize("n_id,n_streams", [(255, 11), (65_281, 10), (65_537, 10), (40_001, 17)])
def test_derive_multi_tiles_per_workgroup(ace, n_id, n_streams):
    """One and two tiles of 256 keys per workgroup (two from 2,560 tiles over a
    launch's streams on a 256-CU device), ragged last tiles, two launches."""
    import torch
    r = np.random.default_rng(n_id)
    rev = r.integers(0, 256, (n_id, 32), dtype=np.uint8)
    streams = [(r.integers(0, 256, k % 65, dtype=np.uint8).tobytes(), bytes(range(3 * k % 65)))
               for k in range(n_streams)]
    print("derive_multi n_id=%d streams=%d" % (n_id, n_streams), flush=True)
    mid = torch.empty((n_streams, n_id, 16), dtype=torch.int32, device="cuda")
    ace.derive_keys_multi(ace.to_device(rev), streams, mid_out=mid)
    pick = np.unique(np.concatenate([np.arange(0, n_id, 97), [0, n_id - 1]]))
    got = mid[:, torch.from_numpy(pick).cuda()].cpu().numpy().view(np.uint32)
    for k, (salt, info) in enumerate(streams):
        want = oracle.hmac_midstates(oracle.derive_keys(rev[pick], salt, info, 8))
        assert np.array_equal(got[k], np.asarray(want).reshape(-1, 16)), k
