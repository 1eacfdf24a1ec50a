"""The fused path at the edges of the forms for launches of few blocks, and bf16 above 2^10: numbers of workers around the groups that encode side by side, numbers
of blocks around the rules that choose them, with and without losses."""
import zlib

import numpy as np
import pytest
import torch

from _util import TOL, as_f64, dev, masks_to_dev, rel_l2, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def b():
    import paper_2310_06993_amd.binding as binding
    return binding


def _workspace(b, L, k):
    n = b.or_workspace_bytes(L, k)
    return torch.empty(n, dtype=torch.uint8, device=dev()) if n else None


def _assert_close(got, want, kind, where):
    """As a whole, and entry by entry, which a block's norm does not show: two bf16 results of the same value are at most one step apart,
    2^-7 of the value, twice that with what their encoded values' roundings add (a step of a few among B, spread over the block); fp32
    results eight times the tolerance's rms."""
    assert rel_l2(got, want) <= TOL[kind], where
    g, w = as_f64(got), as_f64(want)
    rms, step = np.sqrt(np.mean(w * w)), 2.0 ** -6 if kind == "bf16" else 8 * TOL["f32"]
    assert (np.abs(g - w) <= step * (np.abs(w) + rms)).all(), where


@pytest.mark.parametrize("loss", [0.0, 0.02, 0.4])
@pytest.mark.parametrize("k,N,blocks", [(11, 2, 3), (11, 3, 1), (11, 7, 257), (11, 8, 512), (11, 9, 513), (11, 17, 2), (12, 3, 256),
                                        (12, 4, 257), (12, 8, 1), (12, 9, 512), (12, 15, 513), (13, 3, 2), (13, 4, 256), (13, 5, 257),
                                        (13, 255, 1), (14, 5, 3), (14, 6, 128), (14, 7, 129), (14, 33, 1), (15, 1, 2), (15, 6, 3),
                                        (16, 1, 1), (16, 3, 64), (16, 2, 65), (16, 2, 129), (16, 5, 3), (16, 2, 258), (16, 40, 1),
                                        (11, 2, 512), (12, 2, 9), (12, 2, 513), (12, 4, 300), (13, 2, 1), (13, 3, 257),
                                        (11, 1, 5), (12, 1, 512), (13, 1, 3), (12, 8, 300), (12, 9, 257), (12, 12, 768), (12, 7, 769), (13, 6, 256),
                                        (13, 7, 9), (16, 3, 321), (16, 1, 300), (16, 4, 513)])
def test_forms_against_the_oracle(b, orc, k, N, blocks, loss):
    """First, middle and last block against the oracle, and the same bits and the arrival total from the batched call.  loss 0: the
    shortcuts for wavefronts and blocks that have everything; 0.4: hardly a run of 32 entries is whole."""
    B, L = 1 << k, blocks << k
    rng = np.random.default_rng(100 * k + N + blocks)
    gen = torch.Generator(device=dev()).manual_seed(k + N)
    x = torch.randn((N, L), device=dev(), generator=gen).mul_(1e-3).to(torch.bfloat16)
    words = np.full((N, L // 32), 0xFFFFFFFF, dtype=np.uint32)
    if loss > 0.1:
        words &= ~(np.uint32(1) << rng.integers(0, 32, words.shape, dtype=np.uint32))
        words[:, -1] &= np.uint32(0x7FFFFFFF)        # the last entry of all is nobody's
    elif loss:
        words.reshape(N, -1, 8)[rng.random((N, L // 256)) < loss] = 0
    md = masks_to_dev(words)
    seed, base = 0x0FEDCBA987654321, (1 << 33) + 4 * B
    out, cnt = torch.full((L,), float("nan"), dtype=torch.bfloat16, device=dev()), torch.full((L,), 255, dtype=torch.uint8, device=dev())
    ws = _workspace(b, L, k)
    b.or_fused_path_bf16(x, md, N, L, k, seed, base, out, cnt, ws)
    for j in {0, blocks // 2, blocks - 1}:
        part = slice(j * B, (j + 1) * B)
        want, wcnt = orc.fused_path(to_np(x[:, part].contiguous()), np.ascontiguousarray(words[:, j * B // 32:(j + 1) * B // 32]), k,
                                    seed, base + j * B)
        assert np.array_equal(to_np(cnt[part]), wcnt), j
        _assert_close(to_np(out[part]), want, "bf16", j)
    again, cnt2 = torch.full_like(out, float("nan")), torch.full_like(cnt, 255)
    totals = torch.full((1,), -1, dtype=torch.int64, device=dev())
    b.or_fused_path_batched_monitored(b.make_buckets([(x, md, again, cnt2, L, seed, base)]), 1, N, k, True, totals, ws)
    assert torch.equal(again.view(torch.uint8), out.view(torch.uint8)) and torch.equal(cnt2, cnt)
    assert totals.item() == cnt.long().sum().item()


@pytest.mark.parametrize("loss", [0.0, 0.01, 0.4])
@pytest.mark.parametrize("k,N,blocks", [(15, 1, 1), (15, 2, 9), (15, 9, 3), (15, 33, 2), (16, 1, 1), (16, 2, 9), (16, 9, 3), (16, 64, 1), (16, 255, 1)])
def test_fp32_large_blocks_against_the_oracle(b, orc, k, N, blocks, loss):
    """fp32 blocks of 2^15 / 2^16, whose whole workers are summed before the encode: none, some and all of the copies whole."""
    B, L = 1 << k, blocks << k
    rng = np.random.default_rng(100 * k + N + blocks)
    gen = torch.Generator(device=dev()).manual_seed(k + N)
    x = torch.randn((N, L), device=dev(), generator=gen).mul_(1e-3)
    words = np.full((N, L // 32), 0xFFFFFFFF, dtype=np.uint32)
    if loss > 0.1:
        words &= ~(np.uint32(1) << rng.integers(0, 32, words.shape, dtype=np.uint32))
        words[:, -1] &= np.uint32(0x7FFFFFFF)        # the last entry of all is nobody's
    elif loss:
        words[rng.random(N) < 0.5, rng.integers(0, L // 32)] = 0x12345678
    md, seed, base = masks_to_dev(words), 0x0FEDCBA987654321, (1 << 33) + 4 * B
    out, room = torch.full((L,), float("nan"), device=dev()), torch.full((L + 3,), 255, dtype=torch.uint8, device=dev())
    cnt, ws = room[3:], _workspace(b, L, k)
    b.or_fused_path(x, md, N, L, k, seed, base, out, cnt, ws)
    for j in {0, blocks // 2, blocks - 1}:
        part = slice(j * B, (j + 1) * B)
        want, wcnt = orc.fused_path(to_np(x[:, part].contiguous()), np.ascontiguousarray(words[:, j * B // 32:(j + 1) * B // 32]), k,
                                    seed, base + j * B)
        assert np.array_equal(to_np(cnt[part]), wcnt), j
        _assert_close(to_np(out[part]), want, "f32", j)
    again, cnt2 = torch.full((2, L), float("nan"), device=dev()), torch.full((2, L), 255, dtype=torch.uint8, device=dev())
    totals = torch.full((2,), -1, dtype=torch.int64, device=dev())
    b.or_fused_path_batched_monitored(b.make_buckets([(x, md, again[j], cnt2[j], L, seed, base) for j in range(2)]), 2, N, k, False, totals, ws)
    for j in range(2):
        assert torch.equal(again[j].view(torch.uint8), out.view(torch.uint8)) and torch.equal(cnt2[j], cnt), j
        assert totals[j].item() == cnt2[j].long().sum().item(), j


@pytest.mark.parametrize("k,N", [(11, 2), (12, 2), (12, 4), (12, 8), (13, 2), (13, 3), (13, 6), (15, 3), (16, 2), (16, 5)])
def test_bits_do_not_depend_on_the_size_of_the_launch(b, k, N):
    """A shard of blocks of 2^11 and more gives, bit for bit, what its beginning gives as a shard of its own or as a bucket among
    others: numbers of blocks on both sides of every change of form, and two rounds of 256 workgroups."""
    B, sizes = 1 << k, (1, 64, 65, 128, 129, 256, 300, 330, 513) if k > 13 else (1, 65, 256, 257, 512, 513, 768, 769)
    gen = torch.Generator(device=dev()).manual_seed(k + N)
    x = torch.randn((N, sizes[-1] * B), device=dev(), generator=gen).mul_(1e-3).to(torch.bfloat16)
    m = torch.where(torch.rand((N, sizes[-1] * B // 2048), device=dev(), generator=gen) < 0.002, 0, -1).to(torch.int32).repeat_interleave(64, 1)
    seed = 0x55AA55AA12345678

    def alone(L):
        out, cnt = torch.full((L,), float("nan"), dtype=torch.bfloat16, device=dev()), torch.full((L,), 255, dtype=torch.uint8, device=dev())
        b.or_fused_path_bf16(x[:, :L].contiguous(), m[:, :L // 32].contiguous(), N, L, k, seed, 0, out, cnt, _workspace(b, L, k))
        return out.view(torch.uint8), cnt

    want, count = alone(sizes[-1] * B)
    for blocks in sizes[:-1]:
        out, cnt = alone(blocks * B)
        assert torch.equal(out, want[:out.numel()]) and torch.equal(cnt, count[:cnt.numel()]), blocks
    L = 65 * B
    xs, ms = x[:, :L].contiguous(), m[:, :L // 32].contiguous()
    outs, cnts = torch.full((5, L), float("nan"), dtype=torch.bfloat16, device=dev()), torch.full((5, L), 255, dtype=torch.uint8, device=dev())
    totals = torch.full((5,), -1, dtype=torch.int64, device=dev())
    b.or_fused_path_batched_monitored(b.make_buckets([(xs, ms, outs[j], cnts[j], L, seed, 0) for j in range(5)]), 5, N, k, True, totals,
                                      _workspace(b, L, k))
    for j in range(5):
        assert torch.equal(outs[j].view(torch.uint8), want[:2 * L]) and torch.equal(cnts[j], count[:L]), j
        assert totals[j].item() == count[:L].long().sum().item(), j


@pytest.mark.parametrize("kind,k,N,L", [("bf16", 10, 2, 1024), ("bf16", 10, 9, 257 << 10), ("bf16", 10, 16, 256 << 10), ("bf16", 10, 33, 1024 << 10),
                                        ("bf16", 10, 3, 1025 << 10), ("bf16", 9, 17, 50 * 512 + 512), ("bf16", 5, 5, 32), ("bf16", 6, 8, 3 * 1024 + 64),
                                        ("bf16", 7, 255, 1024 + 128), ("f32", 9, 5, 2047 * 512), ("f32", 5, 3, 7 * 1024 + 32), ("f32", 8, 2, 256),
                                        ("f32", 11, 3, 256 << 11), ("f32", 11, 4, 257 << 11), ("f32", 12, 8, 128 << 12), ("f32", 12, 13, 200 << 12),
                                        ("f32", 12, 9, 1 << 12), ("f32", 12, 255, 2 << 12)])
@pytest.mark.parametrize("loss", [0.0, 0.3])
def test_side_by_side_groups_against_the_oracle(b, orc, kind, k, N, L, loss):
    """The same for the groups of the stage-by-stage form: whole tiles and tiles cut short, counts at an odd address."""
    f32, B = kind == "f32", max(1 << k, 1024)
    rng = np.random.default_rng(k * 1000 + N + L)
    gen = torch.Generator(device=dev()).manual_seed(k + N)
    x = torch.randn((N, L), device=dev(), generator=gen).mul_(1e-3).to(torch.float32 if f32 else torch.bfloat16)
    words = np.full((N, L // 32), 0xFFFFFFFF, dtype=np.uint32)
    if loss:
        hit = rng.random(words.shape) < loss
        words[hit] &= ~(np.uint32(1) << rng.integers(0, 32, int(hit.sum()), dtype=np.uint32))
        words[:, -1] &= np.uint32(0x7FFFFFFF)        # the last entry of all is nobody's
    md, seed, base = masks_to_dev(words), 0x0FEDCBA987654321, (1 << 33) + 4 * B
    out, room = torch.full_like(x[0], float("nan")), torch.full((L + 5,), 255, dtype=torch.uint8, device=dev())
    cnt = room[5:]
    (b.or_fused_path if f32 else b.or_fused_path_bf16)(x, md, N, L, k, seed, base, out, cnt, None)
    for lo in {0, L // 2 // B * B, (L - 1) // B * B}:
        part = slice(lo, min(lo + B, L))
        want, wcnt = orc.fused_path(to_np(x[:, part].contiguous()), np.ascontiguousarray(words[:, part.start // 32:part.stop // 32]), k,
                                    seed, base + lo)
        assert np.array_equal(to_np(cnt[part]), wcnt), lo
        _assert_close(to_np(out[part]), want, kind, lo)
    again, cnt2 = torch.full_like(out, float("nan")), torch.full((L,), 255, dtype=torch.uint8, device=dev())
    totals = torch.full((1,), -1, dtype=torch.int64, device=dev())
    b.or_fused_path_batched_monitored(b.make_buckets([(x, md, again, cnt2, L, seed, base)]), 1, N, k, not f32, totals, None)
    assert torch.equal(again.view(torch.uint8), out.view(torch.uint8)) and torch.equal(cnt2, cnt)
    assert totals.item() == cnt2.long().sum().item()


@pytest.mark.parametrize("k,blocks", [(10, 2), (11, 2), (11, 600), (12, 2), (12, 600), (13, 2), (13, 600), (14, 2), (14, 300), (15, 2), (16, 1), (16, 66), (16, 130)])
def test_bf16_subnormals_and_infinities(b, orc, k, blocks):
    """What additions give, where the first stages are a matrix product: subnormal entries count, an infinite entry that arrived makes its
    block infinite or NaN as it does in the oracle, and nothing else.

    u = 2^-133, the lowest bf16.  The inputs are multiples of it up to 127 u, encoded values stay below 2^9 u, where bf16 is spaced 2 u: the
    oracle and the kernel (which may scale after the rounding) each move an encoded value by at most u, i.e. by u / sqrt(3) rms.  A decoded
    value is the mean of 3 with a sum of signs: the two differ by sqrt(2 / 9) u rms, 2.9 u at six times that, and by at most u more for each
    of the results' own roundings."""
    B, L, N, u = 1 << k, blocks << k, 3, 2.0 ** -133
    gen = torch.Generator(device=dev()).manual_seed(50 + k)
    x = torch.randint(-127, 128, (N, L), device=dev(), generator=gen).float().mul_(u).to(torch.bfloat16)
    words = np.full((N, L // 32), 0xFFFFFFFF, dtype=np.uint32)
    words[1, 1::7] = 0x0FFF0FFF
    md, seed, base = masks_to_dev(words), 0x0FEDCBA987654321, (1 << 33) + 4 * B
    out, cnt, enc = torch.empty_like(x[0]), torch.empty(L, dtype=torch.uint8, device=dev()), torch.empty_like(x[0])
    ws = _workspace(b, L, k)

    def both(j):
        part = slice(j * B, (j + 1) * B)
        want, wcnt = orc.fused_path(to_np(x[:, part].contiguous()), np.ascontiguousarray(words[:, j * B // 32:(j + 1) * B // 32]), k, seed, base + j * B)
        assert np.array_equal(to_np(cnt[part]), wcnt)
        wenc = orc.rht_encode(to_np(x[2, part].contiguous()), k, seed, base + j * B)
        return as_f64(to_np(out[part])), as_f64(want), as_f64(to_np(enc[part])), as_f64(wenc)

    def run():
        b.or_fused_path_bf16(x, md, N, L, k, seed, base, out, cnt, ws)
        b.or_rht_encode_bf16(x[2].contiguous(), L, k, seed, base, enc)

    run()
    for j in {0, blocks - 1}:
        got, want, genc, wenc = both(j)
        assert np.abs(want).max() > 40 * u and np.abs(got - want).max() <= 5 * u, j
        assert np.abs(genc - wenc).max() <= 2 * u and (genc != wenc).mean() < 0.02, j      # the other side of a rounding boundary now and then
    x.normal_(generator=gen)
    x[2, 7], x[0, L - 1] = float("inf"), -float("inf")
    run()
    for j in {0, blocks - 1}:
        for got, want in (both(j)[:2], both(j)[2:]):
            assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(got[np.isinf(got)], want[np.isinf(want)]), j
    if blocks > 2:
        assert bool(torch.isfinite(out[B:-B]).all())


# crc32 of results and counts, from the kernel as it was before its exchange through LDS was laid out without bank conflicts
BITS_64K = {(2, 2): 3482775782, (9, 66): 52690716, (3, 259): 2449376446}


@pytest.mark.parametrize("N,blocks", sorted(BITS_64K))
def test_bits_of_the_largest_blocks_stay(b, N, blocks):
    """bf16 blocks of 2^16: the order of the additions, and with it every bit of the results, in each split of a block and in the walk.  A
    rounding of an encoded value that goes the other way changes results by a bf16 step, which no tolerance shows.  Values of
    sixteen binades, blocks and halves of blocks of zeros, runs and single entries lost."""
    k, B, L = 16, 1 << 16, blocks << 16

    def noise(count, salt):   # whole numbers only: the same on every machine
        h = torch.arange(count, device=dev(), dtype=torch.int64) * 0x5851F42D4C957F2D + salt * 0x14057B7EF767814F
        h = (h ^ ((h >> 29) & 0x7FFFFFFFF)) * 0x2545F4914F6CDD1D
        return (h >> 31) & 0xFFFFFFFF

    h = noise(N * L, 1)
    x = ((h & 0x807F) | ((108 + ((h >> 16) & 15)) << 7)).to(torch.int32).to(torch.int16).view(torch.bfloat16).view(N, L)
    x[:, B // 2:B] = 0
    x[:, -B:] = 0
    h = noise(N * L // 32, 2).view(N, -1)
    m = torch.where(h % 97 == 0, h, 0xFFFFFFFF)
    m.view(N, -1, 16)[h.view(N, -1, 16)[:, :, 0] % 31 == 0] = 0
    m[0, 2048 * (blocks // 2):2048 * (blocks // 2 + 1)] = 0xFFFFFFFF
    out, cnt = torch.empty(L, dtype=torch.bfloat16, device=dev()), torch.empty(L, dtype=torch.uint8, device=dev())
    b.or_fused_path_bf16(x, m.to(torch.int32), N, L, k, 0x0123456789ABCDEF, 5 * B, out, cnt, _workspace(b, L, k))
    assert zlib.crc32(to_np(cnt).tobytes(), zlib.crc32(to_np(out).tobytes())) == BITS_64K[N, blocks]
