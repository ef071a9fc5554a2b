"""The divergence check's lists of divergent blocks at the sizes where they
change hands: what the kernels write to host memory and one block more, every
block of a chunk, more chunks than one scan step, counts that start off a
four-word boundary."""
import numpy as np
import pytest

from test_gpu_divergence import ctx, same_as_oracle  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("divergent", [0, 1, 1023, 1024, 1025, 5000])
@pytest.mark.parametrize("tpb", [2, 63, 64, 65, 250])
def test_number_of_blocks(ctx, divergent, tpb):  # noqa: F811
    rng = np.random.default_rng(divergent + tpb)
    n_blocks = 6000
    counts = np.repeat(rng.integers(0, 3, n_blocks), tpb)
    at = rng.permutation(n_blocks)[:divergent].astype(np.int64)
    counts[at * tpb + rng.integers(0, tpb, divergent)] += 5
    print(f"[gpu] {divergent} divergent blocks of {tpb}", flush=True)
    assert len(same_as_oracle(ctx, counts, [0, 1000 * tpb, n_blocks * tpb], [tpb, tpb])) == divergent


@pytest.mark.parametrize("tpb,n_blocks", [(2, 8192), (4097, 7), (20000, 3)])
def test_every_block(ctx, tpb, n_blocks):  # noqa: F811
    counts = np.ones(tpb * n_blocks, dtype=np.uint32)
    counts[::tpb] = 0  # the first thread of every block leaves
    counts[tpb - 1::tpb] = 2
    print(f"[gpu] every block of {tpb} diverges", flush=True)
    assert len(same_as_oracle(ctx, counts, [0, len(counts)], [tpb])) == n_blocks


def test_many_chunks_and_odd_starts(ctx):  # noqa: F811
    """Traces of odd sizes after each other, more than 4096 chunks of threads."""
    rng = np.random.default_rng(1)
    tpb = np.tile([3, 7, 33, 101], 1100).astype(np.uint32)
    blocks = np.tile([5, 1, 9, 45], 1100)
    off = np.concatenate([[0], np.cumsum(blocks * tpb)]).astype(np.uint64)
    counts = np.repeat(rng.integers(0, 4, int(blocks.sum())), np.repeat(tpb, blocks))
    counts[rng.integers(0, len(counts), 900)] += 1
    print("[gpu] 4400 short traces", flush=True)
    assert len(same_as_oracle(ctx, counts, off, tpb)) > 500
