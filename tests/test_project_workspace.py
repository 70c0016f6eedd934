"""Host-side: a projection workspace serves every smaller batch and gradient length of the same projection."""
import random

from paper_2502_01703_amd import binding as Q


def test_workspace_serves_smaller_batches_and_lengths():
    rng = random.Random(5)
    for _ in range(2000):
        k = 64 * rng.choice([1, 8, 42, 52, 128, 256])
        n = rng.randint(1, 1024) if rng.random() < 0.5 else rng.randint(1, 64)
        d = int(2 ** rng.uniform(0, 27))
        most = Q.project_workspace(n, d, k)
        assert most >= n * k * 4
        for n2, d2 in ((rng.randint(1, n), d), (n, rng.randint(1, d)), (rng.randint(1, n), rng.randint(1, d))):
            assert Q.project_workspace(n2, d2, k) <= most, (n, d, k, n2, d2)
