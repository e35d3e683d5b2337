"""GPU parity of the gather's walk over the lanes: lane counts around a whole number of table groups (eight), lanes without a
complete transition among the others, wrapped and unwrapped rings, terminal flags in most windows -- bit-exact vs the oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2111_01264_amd as P
from datagen import synth
from oracle.replay import OracleReplay
from tests.gpu_util import dev
from tests.test_gpu_replay import check_equal, gather_gpu


@pytest.mark.parametrize("lanes", [7, 8, 9, 64])
def test_draws_over_lanes(lanes):
    M, seed = 11, 70 + lanes
    st = torch.cuda.Stream()
    rb = P.replay_create(M * lanes, lanes, M, seed, st, st)
    orc = OracleReplay(M * lanes, lanes, seed)
    rng = np.random.default_rng(lanes)
    try:
        keep = []
        for rnd in range(3):
            for lane in range(lanes):
                # none, fewer than a window, one window, full, by lane; later rounds wrap some of the lanes
                n = int((0, 4, 5, M, 3, 1, 7)[(lane + rnd) % 7])
                if not n:
                    continue
                ids = (np.arange(rnd * M, rnd * M + n, dtype=np.uint64) * np.uint64(lanes) + np.uint64(lane))
                f = synth.frames(seed, synth.STREAM_REPLAY, ids)
                a, r, d = synth.transitions(seed, ids, 6, 0.05, 0.05, 0.15)
                keep.append([dev(v) for v in (f, a, r, d)])
                P.replay_push(rb, lane, *keep[-1], n)
                orc.push(lane, f, a, r, d)
            P.replay_flush(rb, 1)
            orc.flush()
            assert P.replay_num_valid(rb) == orc.num_valid() > 0
            check_equal(gather_gpu(rb, 4 * lanes + 3, rnd), orc.sample_indices(4 * lanes + 3, rnd), orc)
        # every index through idx_in: the valid ones as the oracle assembles them, the others marked
        idx = rng.permutation(M * lanes).astype(np.int64)
        s, s2, a, r, d, got = gather_gpu(rb, idx.size, 0, dev(idx))
        ok = np.array([3 <= i % M <= orc.count[i // M] - 2 for i in idx])
        check_equal([v[ok] for v in (s, s2, a, r, d, got)], idx[ok], orc)
        assert (a[~ok] == -1).all() and not s[~ok].any() and not s2[~ok].any() and not r[~ok].any() and not d[~ok].any()
    finally:
        P.replay_destroy(rb)
