"""How the attention of a decode batch is cut into items (CPU: host arithmetic of the built library).  The program checks for
every batch that the items cover each row's keys exactly once and that every slot is written once, in range and merged."""
import numpy as np
import pytest

from paper_2601_11546_amd import workloads as W
from tests import host_program, test_gpu_joint_items


@pytest.fixture(scope="module")
def cut(tmp_path_factory):
    exe = host_program.build(tmp_path_factory.mktemp("items"), "attention_items")

    def ask(shape, own, prefix=0, members=None, page=16):
        head = (shape.n_q_heads, shape.n_kv_heads, shape.head_dim, page, len(own), prefix, len(own) if members is None else members)
        return host_program.run(exe, " ".join(map(str, (*head, *own))) + "\n")[0]
    return ask


# rows of 60 own keys among which `n_long` have `long` of them, behind a template
@pytest.mark.parametrize("shape,rows,n_long,long,prefix", [
    (W.LLAMA_13B, 60, 10, 8000, 512), (W.LLAMA_13B, 100, 1, 8000, 512), (W.LLAMA_13B, 100, 1, 1500, 512), (W.LLAMA_13B, 200, 2, 8000, 512),
    (W.LLAMA_13B, 60, 60, 1000, 512), (W.LLAMA_13B, 2, 2, 8000, 512), (W.LLAMA_70B, 250, 3, 8000, 768), (W.LLAMA_70B, 250, 100, 3000, 768),
    (W.QWEN_32B_TP2, 200, 5, 4000, 256), (W.LLAMA_70B_TP4, 128, 128, 3000, 256), (W.LLAMA_13B, 200, 2, 8000, 0), (W.LLAMA_13B, 100, 1, 3000, 0),
])
def test_long_rows_are_cut(cut, shape, rows, n_long, long, prefix):
    """No wave walks more than a chunk and a half of the longest chunk length (512 keys), whatever the rest of the batch."""
    own = np.full(rows, 60)
    own[np.random.default_rng(1).permutation(rows)[:n_long]] = long
    slots, longest, *_ = cut(shape, own, prefix)
    assert longest < 768, (slots, longest)


def test_small_batches_behind_a_template_are_cut_finely(cut):
    assert cut(W.LLAMA_13B, [136, 100, 64, 31], 512)[1] <= 96             # chunks of 64 keys
    slots, longest, prefix_item, *_ = cut(W.LLAMA_13B, [83] * 24, 512)
    assert slots > 0 and longest < 96 and prefix_item < 512


def test_batches_that_keep_their_rows_in_sequence(cut):
    """Many waves with much to read balance by themselves; without a template slots are for rows nothing else cuts as finely."""
    for own, prefix in (([1024] * 128, 0), ([1000] * 200, 512), ([400] * 256, 512), ([1500, 1500] + [60] * 22, 0), ([100] * 4, 0)):
        assert cut(W.LLAMA_13B, own, prefix)[0] == 0, (len(own), own[0], prefix)


@pytest.mark.parametrize("seed", range(40))
def test_random_batches_are_covered(cut, seed):
    rng = np.random.default_rng(seed)
    shape = [W.TINY, W.TINY_GQA, W.TINY_G5, W.LLAMA_13B, W.LLAMA_70B, W.QWEN_32B_TP2][seed % 6]
    rows = int(rng.integers(1, 257))
    own = np.exp(rng.uniform(0, np.log(9000 if seed % 3 else 300), rows)).astype(int) + 1
    page = int(rng.choice([8, 16, 64, 256]))
    cut(shape, own, int(rng.integers(0, 4000)) // page * page, int(rng.integers(1, rows + 1)), page)


@pytest.fixture(scope="module")
def joint(tmp_path_factory):
    exe = host_program.build(tmp_path_factory.mktemp("joint"), "joint_items")

    def ask(shape, q, own, prefix, page=16, without_slots=False, groups=1):
        rows = " ".join(f"{a} {b}" for a, b in zip(q, own))
        *cut, other = host_program.run(exe, f"{shape.n_q_heads} {shape.n_kv_heads} {shape.head_dim} {page} {prefix} {groups} {len(q)} {rows}\n")[0]
        return other if without_slots else tuple(cut)
    return ask


def test_prefill_rows_of_a_group_take_joint_items(joint):
    assert joint(W.LLAMA_13B, [120] * 16, [120] * 16, 512) == (15, 15, 0)
    assert joint(W.LLAMA_13B, [120] * 16 + [1] * 100, [120] * 16 + [60] * 100, 512) == (16, 15, 1)   # the decode rows' template beside them
    assert joint(W.LLAMA_13B, [8] * 50, [8] * 50, 512) == (50, 0, 0)              # short requests, few items: two passes
    assert joint(W.LLAMA_13B, [8] * 50 + [1] * 9, [8] * 50 + [30] * 9, 512) == (50, 0, 0)
    assert joint(W.LLAMA_13B, [8] * 250, [8] * 250, 512) == (16, 16, 0)           # the same, enough items to fill the chip
    assert joint(W.LLAMA_13B, [200, 1], [200, 9], 512) == (3, 2, 1)


@pytest.mark.parametrize("shape,n,q,cached,prefix,fused", [
    (W.LLAMA_13B, 16, 32, 2000, 512, False), (W.LLAMA_13B, 16, 32, 0, 512, True), (W.LLAMA_13B, 16, 120, 1000, 512, False),
    (W.LLAMA_13B, 4, 100, 2500, 256, False), (W.LLAMA_13B, 500, 4, 0, 256, False),
    (W.LLAMA_70B, 16, 4, 2000, 512, False), (W.LLAMA_70B, 25, 8, 0, 512, True), (W.LLAMA_70B, 16, 32, 2500, 512, True), (W.LLAMA_70B, 100, 4, 1000, 256, False),
    (W.QWEN_32B, 12, 32, 1000, 256, False), (W.QWEN_32B, 50, 8, 64, 1024, False), (W.LLAMA_70B_TP4, 500, 4, 1000, 256, False),
])
def test_keys_cached_behind_the_template_count(joint, shape, n, q, cached, prefix, fused):
    """A joint item walks its requests' cached keys one request after the other: the two passes are kept where that is the slower."""
    assert (joint(shape, [q] * n, [q + cached] * n, prefix)[1] > 0) == fused


@pytest.mark.parametrize("shape,rows,slots", [(W.LLAMA_13B, 100, 1), (W.LLAMA_13B, 409, 1), (W.LLAMA_13B, 410, 0), (W.LLAMA_70B, 256, 1), (W.LLAMA_70B, 257, 0),
                                              (W.LLAMA_70B_TP4, 1024, 1), (W.LLAMA_70B_TP4, 2000, 0)])
def test_many_decode_rows_keep_the_pass_over_their_template(joint, shape, rows, slots):
    """Beside prefill rows: a second state for every row is dearer than a launch that fills the chip."""
    assert joint(shape, [90] * 16 + [1] * rows, [90] * 16 + [60] * rows, 512)[2] == slots


@pytest.mark.parametrize("shape", test_gpu_joint_items.JOINT_SHAPES.values(), ids=test_gpu_joint_items.JOINT_SHAPES)
def test_the_batch_of_the_device_tests_takes_joint_items(joint, shape):
    more_q, more_own = test_gpu_joint_items.TWO_PASSES
    for batch, slots in ((test_gpu_joint_items.JOINT_BATCH, 0), (test_gpu_joint_items.MIXED_BATCH, 1)):
        q, own, prefix = batch
        tiles, n_joint, in_slots = joint(shape, q, own, prefix)
        assert n_joint > 0 and in_slots == slots
        assert joint(shape, [*q, *more_q], [*own, *more_own], prefix)[1:] == (0, 0)


@pytest.mark.parametrize("shape,q,own,prefix,fused", [
    # 16-bit pools: the template's items are in the one launch either way, so the joint items' length counts against two passes of it
    (W.LLAMA_13B, [90] * 16 + [1] * 100, [90] * 16 + [60] * 100, 512, True), (W.LLAMA_70B, [90] * 16 + [1] * 100, [90] * 16 + [60] * 100, 512, True),
    (W.TINY_GQA, [3] * 3 + [1] * 34, [3] * 3 + [30] * 34, 512, False),
    # beside a long stream of the decode rows' own keys: nearly free
    (W.LLAMA_13B, [70] * 16 + [1] * 184, [70] * 16 + [84] * 184, 512, True), (W.LLAMA_13B, [75] * 8 + [1] * 100, [75] * 8 + [84] * 100, 512, True),
    # too many decode rows for slots: the pass over the template stays
    (W.LLAMA_70B, [30] * 4 + [1] * 300, [30] * 4 + [60] * 300, 256, False),
])
def test_decode_rows_need_the_pass_as_well(joint, shape, q, own, prefix, fused):
    """Joint items save no launch where decode rows of their group keep the pass over the template."""
    assert (joint(shape, q, own, prefix)[1] > 0) == fused


@pytest.mark.parametrize("shape,q,own,prefix,fused", [
    (W.LLAMA_70B, [7] * 8 + [1] * 29, [7] * 8 + [60] * 29, 1024, False), (W.TINY_GQA, [50] * 4 + [1] * 9, [50] * 4 + [100] * 9, 512, False),
    (W.QWEN_32B_TP2, [8] * 5 + [1] * 223, [64] * 5 + [34] * 223, 1024, False), (W.LLAMA_13B, [120] * 60 + [1] * 9, [120] * 60 + [30] * 9, 1024, True),
])
def test_decode_rows_over_quantised_pools_keep_the_pass(joint, shape, q, own, prefix, fused):
    """There the pass over the template is never an item of the one launch: joint items run behind it."""
    assert (joint(shape, q, own, prefix, without_slots=True) > 0) == fused


@pytest.mark.parametrize("shape,q,own,prefix,groups,fused", [
    (W.LLAMA_70B, [24, 33, 35, 30, 28, 26, 30, 31, 35, 20, 24, 33, 35, 30, 28], [235, 460, 130, 300, 28, 26, 30, 231, 35, 20, 324, 33, 35, 30, 28], 768, 3, True),
    (W.LLAMA_13B, [120] * 16 + [4] * 16, [120] * 16 + [1500] * 16, 512, 2, False), (W.LLAMA_13B, [120] * 16 + [90] * 16, [120] * 16 + [90] * 16, 512, 2, True),
])
def test_groups_take_joint_items_together(joint, shape, q, own, prefix, groups, fused):
    """Where one group keeps the pass over its template, joint items of another would run behind it."""
    tiles, n_joint, _ = joint(shape, q, own, prefix, groups=groups)
    assert n_joint == (tiles if fused else 0)


@pytest.mark.parametrize("seed", range(30))
def test_random_mixed_batches_are_covered(joint, seed):
    rng = np.random.default_rng(seed)
    shape = [W.TINY, W.TINY_GQA, W.TINY_G5, W.LLAMA_13B, W.LLAMA_70B, W.QWEN_32B_TP2][seed % 6]
    rows = int(rng.integers(2, 60))
    q = np.where(rng.random(rows) < 0.3, 1, np.exp(rng.uniform(0, np.log(300), rows)).astype(int) + 1)
    page = int(rng.choice([8, 16, 64]))
    joint(shape, q, q + rng.integers(0, 200, rows) * (rng.random(rows) < 0.5), int(rng.integers(1, 20)) * page, page)
