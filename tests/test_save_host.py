"""FlashD2H's host side on the CPU: the saver runs against a stand-in for the
few HIP calls it makes (copies done at once and counted, events that are
always ready), found before the HIP runtime's own, so its copies, its threads
and its scatter are the library's.  Every byte of the pool against the oracle,
and the number of copies: one for a save of less than 4 MiB, whatever the
number of rows left over from whole blocks, at most sqrt(MiB) beyond."""
import json
import math

import hip_stand_in
import pytest

CHILD = r"""
import oracle
c, D = json.loads(sys.argv[2]), 128
B, n_new, Hkv, blk, lens = c["B"], c["n_new"], c["Hkv"], c["blk"], np.asarray(c["lens"], np.int32)
rng = np.random.default_rng(B * 1000 + n_new)
rec = 2 * blk * D * 2
blocks = (int(lens.max()) + c["saves"] * n_new) // blk + 1
pool = np.frombuffer(rng.bytes(B * Hkv * blocks * rec), np.uint8).copy()
want = pool.copy()
off, room = np.arange(B * Hkv, dtype=np.int64) * blocks * rec, np.full(B, blocks, np.int32)
saver = ss.ss_kv_saver_create(B, Hkv, blk, D, pool.ctypes.data, off, room, n_new, 2, c["threads"])
new, copies, impl = [], [], oracle.Oracle()
for s in range(c["saves"]):  # issued one after another: the third waits for the first one's staging buffer
    new.append(rng.integers(0, 1 << 16, (B, n_new, Hkv, 2, D), dtype=np.uint16))
    ss.ss_kv_save(saver, new[s].ctypes.data, n_new, lens + s * n_new, stream=0)
    copies.append(stand_in.stand_in_copies())
ss.ss_kv_save_wait(saver)
ss.ss_kv_saver_destroy(saver)
for s in range(c["saves"]):
    impl.save(new[s], lens + s * n_new, blk, want, off, room)
print(json.dumps({"copies": copies, "equal": bool(np.array_equal(pool, want))}))
"""


@pytest.fixture(scope="module")
def stand_in(tmp_path_factory):
    return hip_stand_in.build(tmp_path_factory.mktemp("stand_in")) or pytest.skip("no C compiler")


@pytest.mark.parametrize("B,n_new,Hkv,blk,lens,threads", [
    (20, 1, 8, 16, [7 * b % 40 for b in range(20)], 2),   # decode steps: a row a sequence
    (11, 1, 4, 8, [b for b in range(11)], 8),
    (33, 1, 8, 32, [31 + b for b in range(33)], 3),
    (1, 1, 1, 16, [15], 1),
    (1, 500, 2, 16, [0], 8),                              # a chunk that ends inside a block
    (3, 17, 8, 16, [0, 3, 20], 2),
    (5, 9, 2, 32, [0, 30, 31, 32, 5], 4),
    (2, 511, 8, 16, [9, 0], 8),                           # just under 4 MiB
    (2, 513, 8, 16, [9, 0], 8),                           # two copies
    (1300, 1, 8, 16, [b % 50 for b in range(1300)], 8),   # two copies of sequences
    (1, 8191, 8, 16, [3], 8)])
def test_copies_and_bytes(stand_in, B, n_new, Hkv, blk, lens, threads):
    size = B * n_new * Hkv * 512
    case = {"B": B, "n_new": n_new, "Hkv": Hkv, "blk": blk, "lens": lens, "threads": threads,
            "saves": 3 if size < (8 << 20) else 1}
    got = json.loads(hip_stand_in.run(stand_in, CHILD, json.dumps(case)))
    assert got["equal"]
    most = max(1, int(math.sqrt(size / (1 << 20))))
    assert all(1 <= n <= most for n in got["copies"]), (got["copies"], most)
