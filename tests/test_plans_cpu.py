"""The launch plans of a step (which workgroup does what), as the step takes
them, over many shapes: no GPU needed."""
import ctypes as C
import random

import pytest

import paper_2405_18628_amd as ppd

CUS = 256


def attention_plan(nh, nkv, Ls, Ts, cus=CUS):
    """(splits, chunk in 32-key blocks, slots of an XCD, splits meet in the kernel)"""
    B = len(Ls)
    I = C.c_int32 * B
    splits, chunk, info = I(), I(), (C.c_int32 * 2)()
    ppd.lib().ppd_plan_attention(nh, nkv, B, I(*Ls), I(*Ts), cus, splits, chunk, info)
    return list(splits), list(chunk), info[0], bool(info[1])


@pytest.mark.parametrize("cus", [CUS, 128])
def test_attention_plan_covers_every_block(cus):
    rng = random.Random(1)
    for _ in range(3000):
        nkv = rng.choice([1, 2, 4, 5, 8, 16, 40])
        nh = nkv * rng.choice([1, 2, 4, 8])
        B = rng.choice([1, 1, 2, 3, 4, 6, 8, 16])
        Ts = [rng.randint(1, 128 // B) for _ in range(B)]
        Ls = [int(2 ** rng.uniform(0, 15)) - 1 for _ in range(B)]
        splits, chunk, slots, meet = attention_plan(nh, nkv, Ls, Ts, cus)
        unit = -(-nh // 8)
        assert slots == unit * sum(splits)
        for L, T, s, c in zip(Ls, Ts, splits, chunk):
            blocks = -(-(L + T) // 32)
            assert 1 <= s <= max(1, min(64, 256 // nh))  # rows of the workspace
            assert (s - 1) * c < blocks <= s * c
        if max(splits) > 1:
            # workgroups wait for each other only where all are resident, and
            # two such launches at once leave compute units for either
            assert not meet or (cus == CUS and slots <= 32)
            assert not meet or B == 1 or max(splits) <= 16
            assert meet or B > 1 or cus != CUS


@pytest.mark.parametrize("nh,nkv,Ls,T", [
    (32, 32, [16384] + [256] * 7, 16),
    (32, 32, [8192] + [300] * 15, 8),
    (32, 8, [16384] + [256] * 7, 16),
    (40, 40, [8192] + [512] * 5, 16),
    (16, 16, [8192] + [300] * 15, 8),
])
def test_a_long_sequence_of_a_batch_is_shared(nh, nkv, Ls, T):
    """The longest run of blocks one compute unit gets, where one sequence
    outweighs the rest of its batch: at most an even share of all blocks and a
    few more (a whole sequence would be 3 to 9 times that)."""
    splits, chunk, slots, meet = attention_plan(nh, nkv, Ls, [T] * len(Ls))
    share = -(-nh // 8) * sum(-(-(L + T) // 32) for L in Ls) / 32
    assert max(chunk) <= max(1.25 * share, 512 / min(64, 256 // nh) + 8)


@pytest.mark.parametrize("nh,nkv,Ls,Ts", [
    (32, 32, [2048], [64]), (16, 16, [200], [16]), (40, 40, [4096], [128]),
    (32, 32, [2048] * 4, [16] * 4), (32, 32, [2048] * 8, [16] * 8), (40, 40, [2048] * 7, [16] * 7),
    (40, 40, [32768, 256], [16, 16]),  # bound by the cache's stream: nothing to balance
])
def test_even_batches_need_no_second_launch(nh, nkv, Ls, Ts):
    splits, _, _, meet = attention_plan(nh, nkv, Ls, Ts)
    assert meet or max(splits) == 1
