"""GPU: plans at the size where a launch's metadata stops fitting its own arguments (3072 bytes) and
is uploaded instead: page chunks of an append (32 bytes each), page ids of an unpack (4), decode
conversations (16, and 4 per work item), extend conversations (16) with their tiles (8 or 16), and
the plans a mixed step hands to its append. Same oracle and tolerance on both sides of the line."""
import numpy as np
import pytest
import torch

from oracle import kvwire
from oracle.attention import attend_last
from synth.values import bf16_bits
from tests.helpers import assert_close, f64, kv_tokens, q_tokens

pytestmark = pytest.mark.gpu

SEED = 909
HQ, HKV, D = 4, 2, 64


def _pool(n_pages, max_convs, layers=1):
    from paper_2606_01839_amd import KVPool
    return KVPool(layers, HQ, HKV, D, n_pages=n_pages, max_convs=max_convs, max_pages_per_conv=1024,
                  placement_seed=4, device="cuda")


@pytest.mark.parametrize("pages", [96, 97, 768, 769])
def test_append_and_unpack_bytes(pages):
    n = 16 * pages - 5
    src, dst = _pool(pages + 2, 2), _pool(pages + 2, 2)
    c = src.conv_create()
    k, v = kv_tokens(SEED, 0, 1, 0, n, HKV, D)
    src.kv_append(c, k.cuda(), v.cuda())
    wire = src.kv_pack(c)
    again = dst.kv_pack(dst.kv_unpack(wire, n))
    torch.cuda.synchronize()
    want = kvwire.serialize(bf16_bits(k), bf16_bits(v))
    assert np.array_equal(wire.cpu().numpy().view(np.uint16), want)
    assert np.array_equal(again.cpu().numpy().view(np.uint16), want)


@pytest.mark.parametrize("ordered", [False, True])
@pytest.mark.parametrize("n", [58, 59, 60, 96, 97, 128, 129, 153, 154])
def test_batches_of_n_conversations(n, ordered):
    """A mixed step of n conversations (extend chunks for the first third, one token each for the
    others), then a decode and an extend batch over all n, one layer of each checked."""
    layers, ne = 2, n // 3
    pool = _pool(6 * n, n, layers)
    lens = [1 + 7 * i % 50 for i in range(n)]
    new = [1 + i % 20 for i in range(ne)] + [1] * (n - ne)
    kv = [kv_tokens(SEED, i, layers, 0, lens[i] + new[i], HKV, D) for i in range(n)]
    convs = [pool.conv_create() for _ in range(n)]
    cat = lambda j, a, b: torch.cat([kv[i][j][:, a(i):b(i)] for i in range(n)], 1).contiguous().cuda()
    pool.kv_append_batch(convs, lens, cat(0, lambda i: 0, lambda i: lens[i]), cat(1, lambda i: 0, lambda i: lens[i]))
    tot = [a + b for a, b in zip(lens, new)]
    q = [q_tokens(SEED, i, 0, lens[i], new[i], HQ, D) for i in range(n)]
    qe, qd = torch.cat(q[:ne]).cuda(), torch.cat(q[ne:]).cuda()
    oe, od = pool.mixed_step(convs[:ne], new[:ne], convs[ne:], cat(0, lambda i: lens[i], lambda i: tot[i]),
                             cat(1, lambda i: lens[i], lambda i: tot[i]), torch.stack([qe] * layers),
                             torch.stack([qd] * layers), layer_ordered=ordered)
    last = torch.cat([x[-1:] for x in q]).cuda()
    dec = pool.attn_decode_batch(convs, 0, last)
    ext = pool.attn_extend(convs, new, 1, torch.cat(q).cuda())
    torch.cuda.synchronize()
    row = 0
    for i in range(n):
        refs = [attend_last(f64(q[i]), f64(kv[i][0][l]), f64(kv[i][1][l])) for l in range(layers)]
        r1 = row + new[i]
        for l in range(layers):
            got = oe[l, row:r1] if i < ne else od[l, i - ne:i - ne + 1]
            assert_close(got, refs[l], f"mixed conv {i} layer {l}")
        assert_close(dec[i:i + 1], refs[0][-1:], f"decode conv {i}")
        assert_close(ext[row:r1], refs[1], f"extend conv {i}")
        row = r1
