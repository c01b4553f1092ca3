"""GPU: calls whose launch metadata goes round the upload ring (8 MiB in four quarters) while launches
that read it are still to be issued."""
import pytest
import torch

from tests.helpers import kv_tokens, q_tokens

pytestmark = pytest.mark.gpu

SEED = 31337


@pytest.mark.parametrize("ordered", [False, True])
def test_mixed_step_of_more_chunks_than_the_ring_holds(ordered):
    """A step that appends 200,200 pages: their chunks (32 bytes each) take four uploads of a quarter, so
    they reach the quarter the ring stood in before them. The step's own plans must still be the ones its
    launches read: outputs equal the separate calls' on the same cache, bit for bit."""
    from paper_2606_01839_amd import KVPool
    n, chunk, d = 2002, 1600, 64
    pool = KVPool(1, 1, 1, d, n_pages=n * chunk // 16 + 256, max_convs=n + 2, max_pages_per_conv=chunk // 16 + 8,
                  placement_seed=3, device="cuda")
    convs = [pool.conv_create() for _ in range(n)]
    dec = [pool.conv_create() for _ in range(2)]
    for i, c in enumerate(dec):
        k, v = kv_tokens(SEED, i, 1, 0, 700, 1, d, device="cuda")
        pool.kv_append(c, k, v)
    k, v = kv_tokens(SEED, 5, 1, 0, n * chunk + 2, 1, d, device="cuda")
    qe = q_tokens(SEED, 6, 0, 0, n * chunk, 1, d, device="cuda")
    qd = q_tokens(SEED, 7, 0, 0, 2, 1, d, device="cuda")
    oe, od = pool.mixed_step(convs, [chunk] * n, dec, k, v, qe[None], qd[None], layer_ordered=ordered)
    assert torch.equal(oe[0], pool.attn_extend(convs, [chunk] * n, 0, qe))
    assert torch.equal(od[0], pool.attn_decode_batch(dec, 0, qd))
    pool.close()
