"""How the stored launch shapes are chosen (host only): one shape for small
covers, and among shapes that are as good hot the best cold one."""
from paper_0912_0947_amd import api, tune


def test_small_covers_share_one_shape():
    """Below 2 MB a kernel takes the same time in every shape to within the
    spread of a measurement: one shape per operation, for every size and k, one
    vector per lane (a header or tail vector is a step of its own otherwise), in
    launch order (runs of blocks start at 128 blocks)."""
    for op in (api.OP_EMBED, api.OP_EXTRACT):
        shapes = [api.tune_get(op, k, n) for k in range(1, 9) for n in (1, 4096, 65537, 786432, tune.RUNS_MIN - 1)]
        assert all(s == shapes[0] for s in shapes) and shapes[0]["order"] == 0, (op, shapes)
        assert shapes[0]["unroll"] == 1 and shapes[0]["blocks_per_cu"] == 0, (op, shapes[0])


def test_choice_between_hot_and_cold():
    hot = {0: 10.0, 1: 10.1, 2: 10.15, 3: 10.3}
    assert tune._choose([0, 1, 2, 3], hot, {0: 20.0, 1: 19.0, 2: 15.0, 3: 10.0}) == 2  # 3 is over 2 % slower hot
    assert tune._choose([0, 1, 2], hot, {0: 20.0, 1: 19.95, 2: 19.9}) == 0  # all tie: the plainest
    assert tune._choose([1, 3], hot, {1: 9.0, 3: 8.95}) == 1


def test_plain_shapes_come_first():
    shapes = tune._shapes((0, 1), tune.ORDERS, (0, 1))
    assert shapes[0] == {"block": 256, "unroll": 1, "blocks_per_cu": 0, "nontemporal": 0, "pack": 0, "order": 0}
    assert len(shapes) == 2 * 2 * 2 * len(tune.CAPS) * len(tune.BLOCKS) * len(tune.UNROLLS)
