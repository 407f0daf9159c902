"""What the planners hand to the launches, over many sizes and without a GPU: every key block in exactly one unit and the
units within the room of the workspace; partial sums and partial maxima within theirs; shapes that exist."""
import numpy as np
import pytest

import hooks as H


@pytest.mark.parametrize("hq,hkv", [(32, 8), (64, 8), (16, 2), (8, 8), (2, 1), (64, 1)])
def test_units_cover_every_key_block_once(hq, hkv):
    rng = np.random.default_rng(hq * 100 + hkv)
    for case in range(200):
        n = 1 + int(rng.integers(1 << int(rng.integers(1, 9)))) if case % 40 else 1 + int(rng.integers(4096))
        top = 1 << int(rng.integers(6, 16))
        keys = [[top] * n, list(rng.integers(1, top + 1, n)), [top] + list(rng.integers(1, 200, n - 1)), [top if i % 2 else 1 + i % 64 for i in range(n)]][case % 4]
        keys = [int(k) for k in keys]
        M = int(rng.integers(1, 66))
        u, splits, room = H.units(keys, M, hq, hkv)
        assert len(u) == sum(splits) <= room and max(splits) <= 512
        i = 0
        for s, k in enumerate(keys):
            at = 0
            for t in range(splits[s]):
                assert u[i][:3] == (s, t, at) and u[i][3] > at
                at, i = u[i][3], i + 1
            assert at == (k + 63) // 64
        # room for the partial results: one a sequence and at most four rounds of the CUs more
        assert sum(splits) <= n + 4 * 256


def test_few_row_plans():
    rng = np.random.default_rng(3)
    for _ in range(2000):
        R, N, K = int(rng.integers(1, 81)), 16 * int(rng.integers(1, 2000)), 128 * int(rng.integers(1, 120))
        for mode in (0, 1, 2):
            pid, splits = H.plan(R, N * 2, K, mode)
            assert mode in H.SHAPE_MODES[pid] and 1 <= splits <= (16 if mode == 0 else 1) and K // 128 % splits == 0


def test_many_row_plans_stay_within_their_buffers():
    rng = np.random.default_rng(4)
    for _ in range(1500):
        R, N, K = int(rng.integers(81, 3000)), 32 * int(rng.integers(1, 1500)), 128 * int(rng.integers(1, 120))
        for mode in (0, 1, 2):
            cap = R * N * int(rng.integers(1, 9))
            head, _ = H.plan(80, N, K, 1)                    # what a model sizes its partial maxima by
            parts = -(-N // H.cols_per_group(head))
            pid, splits = H.plan(R, N, K, mode, part_elems=cap, amax_parts=parts)
            mt, cfg = (pid - H.ROWS) // 4, (pid - H.ROWS) % 4
            assert 4 <= mt <= 8 and cfg in (0, 1, 2)
            chunks = K // (32 * H.CONFIGS[cfg][1])
            assert chunks % splits == 0 and (mode == 0 or splits == 1) and splits * R * N <= cap
            if mode == 1:
                assert -(-N // H.cols_per_group(pid)) <= parts
