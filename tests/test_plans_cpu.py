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


GEMMS = {"qkv": 0, "o": 1, "gate_up": 2, "lm_head": 3, "down": 1}


def gemm_plan(which, hidden, heads, kv, ffn, vocab, T, cus=CUS):
    """(groups of the largest tile, tiles of an XCD, K slices)"""
    N, K = {"qkv": ((heads + 2 * kv) * 128, hidden), "o": (hidden, heads * 128), "gate_up": (ffn, hidden),
            "lm_head": (vocab, hidden), "down": (hidden, ffn)}[which]
    p = (C.c_int32 * 3)()
    ppd.lib().ppd_plan_gemm(GEMMS[which], N, K, T, cus, p)
    return tuple(p)


# Shapes (hidden, heads, kv heads, ffn, vocab) whose GEMMs are split over K, the
# tokens of a step, and the (groups, slices) planned: every kind with 2, 4 and 8
# slices where shapes get them, tiles of 1 to 8 groups, ragged ones among them.
SPLIT_CASES = [
    ((4096, 32, 8, 1024, 500), 33, dict(qkv=(3, 2), o=(4, 4), gate_up=(1, 4), lm_head=(1, 8))),
    ((4096, 4, 4, 2176, 5000), 112, dict(qkv=(3, 8), gate_up=(3, 4), lm_head=(6, 4))),
    ((5120, 8, 8, 1344, 5000), 16, dict(gate_up=(3, 8), lm_head=(3, 2))),
    ((5120, 8, 8, 1344, 700), 75, dict(qkv=(3, 4), gate_up=(3, 8))),
    ((5120, 38, 38, 13056, 300), 50, dict(qkv=(8, 2), o=(6, 4), gate_up=(7, 2), down=(6, 4))),
    ((5120, 38, 2, 12800, 300), 18, dict(o=(6, 4), gate_up=(4, 1), down=(6, 4))),
    ((2048, 40, 40, 1344, 900), 100, dict(qkv=(4, 1), o=(2, 4), gate_up=(1, 2))),
    ((5120, 36, 36, 512, 300), 110, dict(qkv=(8, 2))),
    ((2560, 4, 4, 8192, 100), 128, dict(down=(6, 8))),
    ((1024, 8, 8, 8192, 300), 9, dict(down=(2, 8))),
    ((384, 8, 2, 6912, 300), 80, dict(o=(1, 8), down=(1, 8))),
    ((5120, 40, 40, 13824, 300), 16, dict(o=(3, 2), down=(3, 2))),
]


@pytest.mark.parametrize("shape,T,plans", SPLIT_CASES)
def test_split_cases_are_planned_split(shape, T, plans):
    """The parity cases of split GEMMs reach the splits they are for."""
    for which, want in plans.items():
        gw, _, s = gemm_plan(which, *shape, T)
        assert (gw, s) == want, (which, gw, s)


def test_gemm_plan_covers_every_group():
    rng = random.Random(2)
    for _ in range(4000):
        shape = (128 * rng.randint(1, 64), *rng.choice([(1, 1), (4, 2), (16, 16), (32, 8), (40, 40), (64, 8)]),
                 64 * rng.randint(1, 320), rng.randint(1, 130000))
        T = rng.randint(1, 128)
        for which in GEMMS:
            gw, TX, s = gemm_plan(which, *shape, T)
            rows = {"qkv": (shape[1] + 2 * shape[2]) * 128, "gate_up": shape[3], "lm_head": shape[4]}.get(which, shape[0])
            groups = -(-rows // 16)
            assert TX * gw >= -(-groups // 8)
            assert s in (1, 2, 4, 8) and (s == 1 or TX * s == 32)  # waiting workgroups are resident together
            assert gemm_plan(which, *shape, T, cus=128)[2] == 1


@pytest.mark.parametrize("T", [49, 54, 56, 64])
def test_13b_width_tiles_of_seven_groups(T):
    """13B width with 49 to 64 tokens: QKV's 3.75 and gate/up's 3.38 groups a
    workgroup, run as whole tiles of 4, take 42 and 59.5 us a launch; as two
    slices of 7.5 and 6.75 groups 40 and 58, and the step is not slower than
    with tiles dealt to single waves."""
    shape = (5120, 40, 40, 13824, 32000)
    assert gemm_plan("qkv", *shape, T) == (8, 16, 2)
    assert gemm_plan("gate_up", *shape, T) == (7, 16, 2)
    # the same widths with fewer columns keep whole tiles
    assert gemm_plan("qkv", 3072, 40, 40, 13824, 32000, T) == (4, 32, 1)
    assert gemm_plan("gate_up", 3072, 40, 40, 13824, 32000, T) == (4, 32, 1)
