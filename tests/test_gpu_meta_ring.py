"""GPU: calls whose launch metadata goes round the upload ring (8 MiB in four quarters) while launches
that read it are still to be issued."""
import pytest
import torch

from oracle.attention import attend_last
from tests.helpers import assert_close, f64, kv_tokens, q_tokens

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


def _one_token_convs(n, extra_pages=256):
    """A pool with n empty conversations and two of 700 tokens, and the one token of each of the n."""
    from paper_2606_01839_amd import KVPool
    d = 64
    pool = KVPool(1, 1, 1, d, n_pages=n + extra_pages, max_convs=n + 2, max_pages_per_conv=64, placement_seed=3,
                  device="cuda")
    dec = [pool.conv_create() for _ in range(2)]
    for i, c in enumerate(dec):
        k, v = kv_tokens(SEED, i, 1, 0, 700, 1, d, device="cuda")
        pool.kv_append(c, k, v)
    k, v = kv_tokens(SEED, 5, 1, 0, n + 2, 1, d, device="cuda")
    return pool, [pool.conv_create() for _ in range(n)], dec, k, v


@pytest.mark.parametrize("n", [66_000, 105_000, 125_000])
def test_batch_of_more_tiles_than_the_ring_holds(n):
    """Descriptors (16 bytes) of n conversations travel with every part of their n tiles (16 bytes): 2, 5
    and 18 parts of a quarter of the ring. A query that sees one key gives that key's value exactly."""
    pool, convs, _, k, v = _one_token_convs(n)
    pool.kv_append_batch(convs, [1] * n, k[:, :n].contiguous(), v[:, :n].contiguous())
    q = q_tokens(SEED, 6, 0, 0, n, 1, 64, device="cuda")
    out = torch.full_like(q, float("nan"))
    pool.attn_extend(convs, [1] * n, 0, q, out)
    assert torch.equal(out, v[0, :n])
    pool.close()


@pytest.mark.parametrize("ordered", [False, True])
@pytest.mark.parametrize("n", [66_000, 105_000, 125_000])
def test_mixed_step_of_more_tiles_than_the_ring_holds(n, ordered):
    """The same beside a decode: an extend plan of two parts (two streams), and ones that go round the
    ring (one stream, plans uploaded again)."""
    pool, convs, dec, k, v = _one_token_convs(n)
    q = q_tokens(SEED, 6, 0, 0, n + 2, 1, 64, device="cuda")
    qe, qd = q[:n].contiguous(), q[n:].contiguous()
    oe, od = torch.full_like(qe[None], float("nan")), torch.full_like(qd[None], float("nan"))
    pool.mixed_step(convs, [1] * n, dec, k, v, qe[None], qd[None], oe, od, layer_ordered=ordered)
    assert torch.equal(oe[0], v[0, :n])
    assert torch.equal(od[0], pool.attn_decode_batch(dec, 0, qd))
    pool.close()


@pytest.mark.parametrize("n,hkv", [(129_000, 1), (130_900, 1), (131_055, 1), (131_055, 2)])
def test_long_chunk_beside_descriptors_that_fill_a_quarter(n, hkv):
    """One 1500-row chunk of 3000 tokens, which alone is cut into pieces and 24 merges, in a batch whose
    other conversations have no queries but a descriptor each: up to the largest batch a quarter of the
    ring can describe, where one tile fits beside them."""
    from paper_2606_01839_amd import KVPool
    d, L, c = 64, 3000, 1500
    pool = KVPool(1, 4 * hkv, hkv, d, n_pages=256, max_convs=n, max_pages_per_conv=256, placement_seed=3, device="cuda")
    convs = [pool.conv_create() for _ in range(n)]
    at = n // 2
    k, v = kv_tokens(SEED, 0, 1, 0, L, hkv, d)
    pool.kv_append(convs[at], k.cuda(), v.cuda())
    q = q_tokens(SEED, 0, 0, L - c, c, 4 * hkv, d)
    out = pool.attn_extend(convs, [c if i == at else 0 for i in range(n)], 0, q.cuda())
    assert_close(out, attend_last(f64(q), f64(k[0]), f64(v[0])), f"{n} descriptors")
    pool.close()
