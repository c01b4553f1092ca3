"""GPU: extend and prefill launches whose tiles are cut into pieces of keys (few tiles, long contexts),
against the fp64 oracle and bit for bit against a second run on other pages. The sizes put piece
boundaries inside the diagonal (rows that see no key of a piece), leave a last piece of one key tile
and one key, mix cut and whole tiles, and cover one to 256 query rows of a tile per head shape."""
import numpy as np
import pytest
import torch

from oracle.attention import attend_last
from tests.helpers import assert_close, f64, kv_tokens, q_tokens

pytestmark = pytest.mark.gpu

SEED = 4711
SHAPES = [(32, 8, 128), (16, 8, 128), (64, 8, 128), (8, 8, 128), (2, 1, 128), (4, 2, 64), (32, 8, 64), (16, 2, 64), (4, 4, 64)]


def _run(hq, hkv, d, prefixes, chunks, pool_seed, kv, q, turn1):
    from paper_2606_01839_amd import KVPool
    pool = KVPool(1, hq, hkv, d, n_pages=sum((p + c + 15) // 16 for p, c in zip(prefixes, chunks)) + 8, max_convs=16,
                  max_pages_per_conv=2048, placement_seed=pool_seed, device="cuda")
    convs = []
    for k, v in kv:
        convs.append(pool.conv_create())
        pool.kv_append(convs[-1], k.cuda(), v.cuda())
    out = (pool.attn_prefill_turn1 if turn1 else pool.attn_extend)(convs, chunks, 0, q)
    torch.cuda.synchronize()
    pool.close()
    return out


@pytest.mark.parametrize("hq,hkv,d", SHAPES)
@pytest.mark.parametrize("prefixes,chunks", [
    ([4000], [1]), ([4095], [2]), ([5000], [65]), ([100], [1437]), ([0], [1437]), ([3000], [300]),
    ([2000, 10, 1300, 0], [40, 130, 7, 64]),
], ids=str)
def test_cut_tiles_match_oracle(hq, hkv, d, prefixes, chunks):
    kv = [kv_tokens(SEED, i, 1, 0, p + c, hkv, d) for i, (p, c) in enumerate(zip(prefixes, chunks))]
    q = torch.cat([q_tokens(SEED, i, 0, p, c, hq, d) for i, (p, c) in enumerate(zip(prefixes, chunks))])
    turn1 = not any(prefixes)
    out = _run(hq, hkv, d, prefixes, chunks, 5, kv, q.cuda(), turn1)
    assert torch.equal(out, _run(hq, hkv, d, prefixes, chunks, 6, kv, q.cuda(), turn1))
    row = 0
    for i, c in enumerate(chunks):
        # the oracle's last rows, enough to cover every piece and the chunk's first and last tile
        rows = np.unique(np.r_[0:min(c, 40), max(0, c - 40):c, np.linspace(0, c - 1, 40).astype(int)])
        k, v = f64(kv[i][0][0]), f64(kv[i][1][0])
        for r in rows:
            ref = attend_last(f64(q[row + r:row + r + 1]), k[:prefixes[i] + r + 1], v[:prefixes[i] + r + 1])
            assert_close(out[row + r:row + r + 1], ref, f"conv {i} row {r}")
        row += c


@pytest.mark.parametrize("ordered", [False, True])
@pytest.mark.parametrize("hq,hkv,d", [(16, 8, 128), (32, 8, 64)])
def test_mixed_step_with_cut_tiles_equals_separate_calls(hq, hkv, d, ordered):
    """More layers than the records of one launch have room for (several launches of layers), cut
    extend tiles beside split and single-item decodes: the separate calls' outputs, bit for bit."""
    from paper_2606_01839_amd import KVPool
    layers = 24
    for dec_lens in ([2100, 700], [30, 500]):
        lens, new = [2500] + dec_lens, [90] + [1] * len(dec_lens)
        a, b = (KVPool(layers, hq, hkv, d, n_pages=400, max_convs=4, max_pages_per_conv=200, placement_seed=8)
                for _ in range(2))
        ha, hb = ([p.conv_create() for _ in lens] for p in (a, b))
        kv = [kv_tokens(SEED, i, layers, 0, n + m, hkv, d, device="cuda") for i, (n, m) in enumerate(zip(lens, new))]
        for i, n in enumerate(lens):
            for p, h in ((a, ha), (b, hb)):
                p.kv_append(h[i], kv[i][0][:, :n].contiguous(), kv[i][1][:, :n].contiguous())
        k, v = (torch.cat([x[j][:, n:] for x, n in zip(kv, lens)], 1).contiguous() for j in (0, 1))
        qe = torch.stack([q_tokens(SEED, 0, l, lens[0], 90, hq, d, device="cuda") for l in range(layers)])
        qd = torch.stack([torch.cat([q_tokens(SEED, i, l, lens[i], 1, hq, d, device="cuda") for i in (1, 2)])
                          for l in range(layers)])
        oe, od = a.mixed_step(ha[:1], [90], ha[1:], k, v, qe, qd, layer_ordered=ordered)
        b.kv_append_batch(hb, new, k, v)
        for l in range(layers):
            assert torch.equal(oe[l], b.attn_extend(hb[:1], [90], l, qe[l])), l
            assert torch.equal(od[l], b.attn_decode_batch(hb[1:], l, qd[l])), l
        a.close()
        b.close()


@pytest.mark.parametrize("hq,hkv,d", [(32, 8, 128), (8, 1, 64), (8, 8, 128), (4, 2, 128)])
@pytest.mark.parametrize("lens", [[1025], [2047], [6000], [24571], [1100, 4096, 2500], [1500, 900]], ids=str)
def test_decode_filling_splits_match_oracle(hq, hkv, d, lens):
    """Decode batches small enough to get splits of 32, 64 or 96 keys (and one that keeps its plan: it
    holds a conversation of one item), with and without the allocation-free entry point; 96 items a
    conversation where few kv heads leave room, more than the merge loads ahead."""
    from paper_2606_01839_amd import KVPool
    pool = KVPool(1, hq, hkv, d, n_pages=sum((n + 15) // 16 for n in lens) + 8, max_convs=4, max_pages_per_conv=2048,
                  placement_seed=2, device="cuda")
    kv = [kv_tokens(SEED, i, 1, 0, n, hkv, d) for i, n in enumerate(lens)]
    convs = [pool.conv_create() for _ in lens]
    for c, (k, v) in zip(convs, kv):
        pool.kv_append(c, k.cuda(), v.cuda())
    q = torch.cat([q_tokens(SEED, i, 0, n - 1, 1, hq, d) for i, n in enumerate(lens)])
    out = pool.attn_decode_batch(convs, 0, q.cuda())
    assert torch.equal(out, pool.attn_decode_batch_noalloc(convs, 0, q.cuda(), torch.empty_like(out)))
    for i in range(len(lens)):
        assert_close(out[i:i + 1], attend_last(f64(q[i:i + 1]), f64(kv[i][0][0]), f64(kv[i][1][0])), f"conv {i}")
    pool.close()


@pytest.mark.parametrize("hq,hkv", [(8, 8), (16, 8), (32, 8), (64, 8), (16, 2)])
def test_head_dim_64_two_workgroups_a_cu(hq, hkv):
    """A head_dim 64 launch of more than 640 workgroups takes the form without operand read-ahead. Its
    first conversations alone stay below that and uncut (257 to 320 tiles at 2 kv heads, 65 to 80 at 8),
    in the form that reads ahead: every row the same bits, and on other pages; sampled rows against the
    oracle."""
    d, tile, per = 64, 256 // (hq // hkv), 256 // hkv
    first = [int(1.6 * per) * tile + 17, int(0.7 * per) * tile + 1]
    lens = first + [per * tile + 3]
    wg = [hkv * sum((n + tile - 1) // tile for n in x) for x in (first, lens)]
    assert 512 < wg[0] <= 640 < wg[1]
    kv = [kv_tokens(SEED, i, 1, 0, n, hkv, d, device="cuda") for i, n in enumerate(lens)]
    q = torch.cat([q_tokens(SEED, i, 0, 0, n, hq, d, device="cuda") for i, n in enumerate(lens)])
    out = _run(hq, hkv, d, [0] * 3, lens, 5, kv, q, True)
    rows = sum(first)
    assert torch.equal(out, _run(hq, hkv, d, [0] * 3, lens, 6, kv, q, True))
    assert torch.equal(out[:rows], _run(hq, hkv, d, [0] * 2, first, 7, kv[:2], q[:rows].contiguous(), True))
    row = 0
    for i, n in enumerate(lens):
        k, v = f64(kv[i][0][0]), f64(kv[i][1][0])
        for r in np.unique(np.r_[0:3, np.linspace(0, n - 1, 12).astype(int)]):
            ref = attend_last(f64(q[row + r:row + r + 1]), k[:r + 1], v[:r + 1])
            assert_close(out[row + r:row + r + 1], ref, f"conv {i} row {r}")
        row += n


def _mixed_equals_separate(hq, hkv, d, layers, prefix, chunk, dec_lens, ordered):
    """A mixed step of one chunk and the decoding conversations, and the separate calls on a second
    pool: the same bits; sampled extend rows of the last layer against the oracle."""
    from paper_2606_01839_amd import KVPool
    lens, new = [prefix] + dec_lens, [chunk] + [1] * len(dec_lens)
    pages = sum((n + m + 15) // 16 for n, m in zip(lens, new)) + 8
    a, b = (KVPool(layers, hq, hkv, d, n_pages=pages, max_convs=len(lens), max_pages_per_conv=max(lens) // 16 + 80,
                   placement_seed=s) for s in (8, 9))
    ha, hb = ([p.conv_create() for _ in lens] for p in (a, b))
    new_kv = []
    for i, (n, m) in enumerate(zip(lens, new)):
        k, v = kv_tokens(SEED, i, layers, 0, n + m, hkv, d, device="cuda")
        for p, h in ((a, ha), (b, hb)):
            p.kv_append(h[i], k[:, :n].contiguous(), v[:, :n].contiguous())
        new_kv.append((k[:, n:].clone(), v[:, n:].clone()))
        if i == 0:
            k_ext, v_ext = f64(k[-1]), f64(v[-1])
    k, v = (torch.cat([x[j] for x in new_kv], 1).contiguous() for j in (0, 1))
    qe = torch.stack([q_tokens(SEED, 0, l, prefix, chunk, hq, d, device="cuda") for l in range(layers)])
    qd = torch.stack([torch.cat([q_tokens(SEED, i + 1, l, n, 1, hq, d, device="cuda") for i, n in enumerate(dec_lens)])
                      for l in range(layers)])
    oe, od = a.mixed_step(ha[:1], [chunk], ha[1:], k, v, qe, qd, layer_ordered=ordered)
    b.kv_append_batch(hb, new, k, v)
    for l in range(layers):
        assert torch.equal(oe[l], b.attn_extend(hb[:1], [chunk], l, qe[l])), l
        assert torch.equal(od[l], b.attn_decode_batch(hb[1:], l, qd[l])), l
    for r in np.unique(np.linspace(0, chunk - 1, 20).astype(int)):
        ref = attend_last(f64(qe[-1, r:r + 1]), k_ext[:prefix + r + 1], v_ext[:prefix + r + 1])
        assert_close(oe[-1, r:r + 1], ref, f"row {r}")
    a.close()
    b.close()


@pytest.mark.parametrize("prefix,chunk", [(1200, 300), (1500, 500)])
def test_chained_tiles_two_workgroups_a_cu(prefix, chunk):
    """All layers of an overlapped head_dim 64 step in launches of more than 640 workgroups whose cut
    tiles hold their pieces."""
    _mixed_equals_separate(32, 8, 64, 24, prefix, chunk, [2100, 700], False)


@pytest.mark.parametrize("hq,hkv,d", [(32, 8, 128), (16, 8, 128), (32, 8, 64)])
def test_chained_tiles_in_layer_order(hq, hkv, d):
    """A layer's launch beside a decode large enough that one workgroup takes a cut tile's pieces."""
    _mixed_equals_separate(hq, hkv, d, 2, 1200, 300, [8000] * 12, True)
