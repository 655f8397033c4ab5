"""GPU parity of the server for more than 128 workers (their tables built in
batches of at most 16 groups of 8) and for chunk lengths that are not a multiple
of 4, at the edges of the batches and of the chunk geometries, and of the plain
server that the narrow chunks of both keep.  Every state, packed word and scale
is compared with the oracle after every step, bit for bit (-0 == +0): the
server's sums are exact, so the split into batches may change no bit."""
import pytest

from synth import configs as C

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


BATCHES = [
    # (segments, chunk, W): LD lanes per chunk, groups per batch x batches of the
    # tables; small launches take the plain server
    ([9000, 1024, 1000, 4], 1024, 129),      # plain, 256 lanes
    ([5000, 300], 260, 256),                 # plain, 128 lanes
    ([6000, 2048, 2044], 2048, 136),         # plain, 512 lanes
    ([8192, 4096, 100], 4096, 192),          # LD128, 12 x 2
    ([8192, 8192, 8000], 8192, 257),         # LD256, 12 x 3, one worker in the last group
    ([32768, 16384, 12], 16384, 250),        # LD512, 16 x 2
    ([700, 64, 36], 32, 140),                # plain, 8 lanes
    ([3000, 256, 252], 256, 130),            # plain, 64 lanes
    ([9000, 1020, 4], 1021, 200),            # unaligned, plain
    ([20000, 3000], 4099, 160),              # unaligned: LD256, 10 x 2
    ([34000, 16380], 16383, 129),            # unaligned: LD512, 10 x 2
    ([700, 64, 36], 33, 140),                # unaligned, plain
    ([5000, 1000], 257, 20),                 # unaligned, plain
    ([9000, 2500], 2049, 33),                # unaligned, plain
]


@pytest.mark.parametrize("segs,chunk,world", BATCHES, ids=[f"C{c}-W{w}" for _, c, w in BATCHES])
def test_server_batches(torch_cuda, segs, chunk, world):
    import harness
    wl = C.Workload(name=f"batches-C{chunk}", seg_off=C.offsets(segs), world=world, chunk=chunk,
                    steps=4, tv=[0, 2], tu=[1, 2, 3], gammas=[1e-4] * 4, sigma_g=1e-3)
    report, inexact = harness.run_parity(wl, log=lambda m: print(m, flush=True))
    for t, bad in enumerate(report):
        assert not bad, f"mismatch after step {t - 1}: {bad}"
    assert inexact == 0


# Shards past the size up to which few workers take the plain server (1.5M
# elements, or 16M elements times workers): the tables at every lane count.
PAST_PLAIN = [
    ([1600000, 100, 36], 4, 3), ([1600000, 64], 60, 9), ([1100000, 300], 128, 16),
    ([1600000, 1000], 252, 4), ([1600000, 508], 512, 8), ([1100000, 4000], 1024, 16),
    ([1600000, 3000], 2048, 5), ([1600000, 9000], 4096, 2), ([1100000, 5000], 1500, 16),
]


@pytest.mark.parametrize("segs,chunk,world", PAST_PLAIN,
                         ids=[f"C{c}-W{w}" for _, c, w in PAST_PLAIN])
def test_tables_past_the_plain_sizes(torch_cuda, segs, chunk, world):
    test_server_batches(torch_cuda, segs, chunk, world)


# The same for more than 128 workers and for unaligned chunks, past the sizes up to
# which they take the plain server: groups per batch x batches, or groups.
PAST_PLAIN_MANY = [
    ([900000, 300], 260, 190),               # LD16, 16 x 2
    ([1600000, 1000], 1024, 200),            # LD32, 16 x 2
    ([2200000, 1000], 1024, 129),            # LD32, 16 x 2, one worker in the second
    ([1000000, 2044], 2048, 136),            # LD64, 10 x 2
    ([700000, 100], 2048, 200),              # LD64, 14 x 2
    ([9000, 4096, 100], 4096, 208),          # LD128, 14 x 2
    ([900000, 300], 263, 190),               # unaligned: LD16, 16 x 2
    ([1600000, 1000], 1021, 200),            # unaligned: LD32, 16 x 2
    ([700000, 100], 2047, 200),              # unaligned: LD64, 14 x 2
    ([9000, 4096, 100], 4095, 180),          # unaligned: LD128, 12 x 2
]
PAST_PLAIN_UNALIGNED = [
    ([1300000, 300], 301, 8),                # LD16, 1
    ([1300000, 300], 301, 14),               # LD16, 2
    ([1000000, 300], 301, 60),               # LD16, 8
    ([2200000, 1000], 1001, 5),              # LD32, 1
    ([1700000, 1000], 1022, 32),             # LD32, 4
    ([1700000, 1000], 1001, 100),            # LD32, 16
    ([1300000, 1100], 1101, 3),              # LD64, 1
    ([1900000, 1500], 1501, 20),             # LD64, 3
    ([1700000, 3000], 3001, 12),             # LD128, 2
    ([300000, 2048], 2049, 90),              # LD128, 12
    ([20000, 4096], 4099, 16),               # LD256, 2
    ([20000, 8192], 8190, 60),               # LD256, 8
    ([2150000, 8192], 8191, 4),              # LD256, 1
    ([2150000, 8192], 16383, 3),             # LD512, 1
    ([40000, 16384], 12345, 30),             # LD512, 4
]


# The plain server of unaligned chunks of two and four blocks per lane, and the
# tables past its worker counts.
PLAIN_LONG = [
    ([9000, 4096, 100], 4099, 1), ([30000, 4100], 4101, 8), ([9000, 8192], 8190, 7),
    ([30000, 8196], 8193, 4), ([30000, 12], 12345, 2), ([70000, 16380, 4], 16382, 4),
    ([30000, 4100], 4101, 9), ([30000, 8196], 8193, 5),
]


@pytest.mark.parametrize("segs,chunk,world", PLAIN_LONG,
                         ids=[f"C{c}-W{w}" for _, c, w in PLAIN_LONG])
def test_plain_server_of_long_unaligned_chunks(torch_cuda, segs, chunk, world):
    test_server_batches(torch_cuda, segs, chunk, world)


@pytest.mark.parametrize("segs,chunk,world", PAST_PLAIN_MANY,
                         ids=[f"C{c}-W{w}" for _, c, w in PAST_PLAIN_MANY])
def test_batches_past_the_plain_sizes(torch_cuda, segs, chunk, world):
    test_server_batches(torch_cuda, segs, chunk, world)


@pytest.mark.parametrize("segs,chunk,world", PAST_PLAIN_UNALIGNED,
                         ids=[f"C{c}-W{w}" for _, c, w in PAST_PLAIN_UNALIGNED])
def test_unaligned_tables_past_the_plain_sizes(torch_cuda, segs, chunk, world):
    test_server_batches(torch_cuda, segs, chunk, world)
