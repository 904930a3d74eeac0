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
