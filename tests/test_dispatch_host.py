"""Which launches the library's host code makes, and which calls it refuses,
on the CPU with a stand-in for HIP (hip_stand_in): sizes at the limits that
no GPU has the memory for, and buffers of every size that is accepted."""
import json

import hip_stand_in
import pytest


@pytest.fixture(scope="module")
def stand_in(tmp_path_factory):
    return hip_stand_in.build(tmp_path_factory.mktemp("stand_in")) or pytest.skip("no C compiler")


ATTENTION = r"""
G, P, got = 4, 0x1000, []
for units, k, blk in json.loads(sys.argv[2]):
    one = units * G * 130 * 4  # bytes of one split's partials
    steps = -(-k * blk // 16)
    n = max(1, min(-(-512 // units), steps // 16))
    need = -(-steps // -(-steps // n)) * one if n > 1 else 0  # the least that was ever asked for
    query = ss.ss_sparse_attention_workspace(units, G, 1, 128, blk, k)
    def call(size):
        ss.ss_sparse_attention(P, P, P, P, None, k, units, G, 1, 128, blk, k, 0.1, P, P if size else None, size, stream=0)
        return launches()
    refused = None
    if need:
        try:
            call(need - 1)
        except ss.SparseServeError as e:
            refused = e.status == ss.SS_ERR_OOM
        assert launches() == []
    got.append({"units": units, "one": one, "need": need, "query": query, "refused": refused, "least": call(need),
                "between": call((need + query) // 2), "full": call(query)})
print(json.dumps(got))
"""


def test_attention_takes_every_workspace_size(stand_in):
    """Two 4-wave workgroups a CU of 16 steps or more each are the partials
    that a caller has always had to bring: a workspace of that size is enough
    for every shape, one byte less is refused, and whatever lies between it
    and what the query asks for holds the partials of the launch it gets."""
    shapes = [(u, s, 16) for u in (1, 2, 4, 8, 9, 16, 24, 32, 44, 64, 95, 100, 143, 200, 256, 257, 320, 341, 384, 511,
                                   512, 1000) for s in (1, 15, 31, 32, 33, 47, 64, 100, 128, 256, 511)]
    shapes += [(8, 512, 8), (2, 65, 8), (3, 128, 32)]
    fewer = 0
    for c in json.loads(hip_stand_in.run(stand_in, ATTENTION, json.dumps(shapes))):
        assert c["query"] >= c["need"] and c["refused"] is not False, c
        for size, made in ((c["need"], c["least"]), ((c["need"] + c["query"]) // 2, c["between"]),
                           (c["query"], c["full"])):
            units, splits = made[0][:2]
            assert units == c["units"] and len(made) == (2 if splits > 1 else 1), c
            assert splits == 1 or splits * c["one"] <= size, c
        assert c["least"][0][1] <= c["between"][0][1] <= c["full"][0][1], c
        fewer += c["least"][0][1] < c["full"][0][1]
    assert fewer > 10  # the shapes reach plans with more splits than the least size holds


SPLITS = r"""
P, got = 0x1000, []
for B, Hq, Hkv, blk, k in json.loads(sys.argv[2]):
    n = ss.ss_sparse_attention_workspace(B, Hq, Hkv, 128, blk, k)
    ss.ss_sparse_attention(P, P, P, P, P, 300, B, Hq, Hkv, 128, blk, k, 0.1, P, P if n else None, n, stream=0)
    got.append(launches())
print(json.dumps(got))
"""


def test_shapes_of_the_scratch_tests_split(stand_in):
    """The shapes that test_zz_no_alloc.py runs to fill the static scratch,
    which takes the plan of its full workspace: a launch of units x splits
    workgroups and the merge; and the one that runs without."""
    made = json.loads(hip_stand_in.run(stand_in, SPLITS, json.dumps([(2, 32, 8, 16, 128), (1, 8, 2, 16, 64),
                                                                     (64, 32, 8, 16, 8)])))
    assert [x[0][:2] for x in made] == [[16, 16], [2, 16], [512, 1]] and [len(x) for x in made] == [2, 2, 1], made


SCORE = r"""
P, got = 0x1000, []
for B, Hkv, n in json.loads(sys.argv[2]):
    made = {}
    for name, call in (("score", lambda: ss.ss_score_blocks(P, P, P, B, Hkv, Hkv, n, 128, P, stream=0)),
                       ("mean", lambda: ss.ss_score_blocks_variant(P, P, 1, 1, P, B, Hkv, Hkv, n, 128, P, stream=0)),
                       ("topk", lambda: ss.ss_score_topk(P, P, P, B, Hkv, Hkv, n, 128, 4, P, P, stream=0))):
        try:
            call()
            made[name] = launches()
        except ss.SparseServeError as e:
            assert e.status == ss.SS_ERR_UNSUPPORTED and launches() == []
            made[name] = None
    got.append(made)
print(json.dumps(got))
"""


@pytest.mark.parametrize("B,Hkv,n,taken", [
    (1, 1, 1, True), (64, 8, 8192, True), (512, 8, 128, True),
    (1 << 19, 8, 256, True), (1, 1 << 22, 256, True),    # 2^22 units of eight score workgroups: more than one launch
    (1 << 20, 8, 100, True), (3, 1 << 21, 129, True),
    ((1 << 21) - 1, 8, 16, True),
    (1 << 20, 1 << 12, 16, False), (1 << 21, 8, 16, False), (1 << 12, 1 << 20, 128, False),  # 2^32, 2^24 units
    (1 << 15, 8, 65536, False)])
def test_score_launch_limits(stand_in, B, Hkv, n, taken):
    """Scoring takes up to 2^32 - 1 threads' worth of 256-block pieces, as it
    always has, in as many launches as the smaller pieces of today need, none
    of them past the 2^32 - 1 threads of a launch; more is refused, by
    ss_score_topk for short rows too."""
    made = json.loads(hip_stand_in.run(stand_in, SCORE, json.dumps([(B, Hkv, n)])))[0]
    units = B * Hkv
    for name, shapes in made.items():
        assert (shapes is not None) == taken, (name, shapes)
        if taken:
            assert all(0 < x * threads < 1 << 32 for x, _, _, threads in shapes), (name, shapes)
            if name != "topk":
                blocks = {128: 32, 256: 256}[shapes[0][3]]  # a workgroup's
                assert sum(x for x, _, _, _ in shapes) == units * (-(-n // blocks)), (name, shapes)
            else:
                assert shapes[-1][0] == units, shapes


METADATA = r"""
P, got = 0x1000, []
for B, Hkv, n, blk, row in json.loads(sys.argv[2]):
    made = []
    for kind in (0, 1):
        try:
            ss.ss_build_metadata_strided(P, P, P, B, Hkv, n, blk, 128, blk * row, row, kind, P, stream=0)
            made.append(launches())
        except ss.SparseServeError as e:
            assert e.status == ss.SS_ERR_UNSUPPORTED and launches() == []
            made.append(None)
    got.append(made)
print(json.dumps(got))
"""


@pytest.mark.parametrize("B,Hkv,n,blk,row,cuboid,mean", [
    (1, 1, 1, 8, 256, True, True), (1, 8, 8192, 16, 4096, True, True),
    (1 << 25, 8, 1, 8, 256, True, False),                # 2^28 blocks of 8: eight of them a wave, whatever the units
    (1 << 22, 8, 3, 16, 256, True, False), (1 << 22, 8, 1, 32, 256, True, True),
    (1 << 13, 8, 65, 8, 4096, True, True), (1 << 20, 8, 61, 8, 4096, True, False),
    ((1 << 29) - 32, 1, 1, 8, 256, True, False), (1 << 29, 1, 1, 8, 256, False, False)])
def test_metadata_launch_limits(stand_in, B, Hkv, n, blk, row, cuboid, mean):
    """Metadata takes what 2^32 - 1 threads of 64/blk blocks (mean keys: one)
    a wave hold, however short the units' rows are, in one launch."""
    made = json.loads(hip_stand_in.run(stand_in, METADATA, json.dumps([(B, Hkv, n, blk, row)])))[0]
    for shapes, taken in zip(made, (cuboid, mean)):
        assert (shapes is not None) == taken, shapes
        if taken:
            (x, _, _, threads), = shapes
            assert 0 < x * threads < 1 << 32
