"""The block-sorted form of the binned insertion at the sizes where its plan
changes, every output bit-exact against the oracle: block edges, the small and
the large blocks, one and two hashing workgroups per CU, the largest countBF
it takes and the next one, short and long runs, every held-cell count of the
region pass, several hash functions and two-word keys."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_2305_07545_amd")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle.build(force=False)
    P.load_library()


def reads_of(seed, n_bases, k):
    """Ragged reads of exactly n_bases bases, with a few 'N', half of them twice."""
    a = synth.random_reads(seed, max(1, n_bases // 300), 40, 260, k=k, p_n=0.003)
    a = synth.concat_reads([a, a, a])
    assert a.n_bases >= n_bases
    offs = a.offsets[a.offsets < n_bases]
    offs = np.append(offs, np.uint64(n_bases))
    return synth.ReadSet("blocks", a.reads[:n_bases].copy(), offs, k, 2, 1.0)


# (bases, X, Y, alpha, k_h, k): words / (cells per region) = regions
CASES = [
    (4095, 269, 281, 8, 1, 21), (4096, 269, 281, 8, 1, 21), (4097, 269, 281, 8, 1, 21),
    (70_001, 3, 5, 8, 1, 31),                 # one region: one run per block
    (300_000, 601, 607, 4, 1, 25),            # 16 counters a cell, 1024 cells a region
    (300_000, 601, 607, 5, 2, 25),            # 12 counters a cell
    (300_000, 601, 607, 16, 3, 25),           # 4 counters a cell
    (300_000, 601, 607, 32, 1, 25),           # 2 counters a cell
    (300_000, 601, 607, 3, 5, 25),            # 21 counters a cell: 512 cells a region
    (200_003, 1009, 1013, 8, 8, 55),          # two-word keys, eight hash functions
    (500_000, 2707, 2711, 8, 1, 31),          # 3584 regions
    (500_000, 2709, 2711, 8, 1, 31),          # 3587 regions
    (500_000, 3829, 3833, 8, 1, 40),          # 7167 regions
    (500_000, 3833, 3837, 8, 1, 31),          # 7182 regions: two-level form
    (8_388_607, 809, 811, 8, 1, 31), (8_388_608, 809, 811, 8, 1, 31),  # small | large blocks
    (8_400_001, 2709, 2711, 8, 1, 31),        # blocks of 32768
]


@pytest.mark.parametrize("n,X,Y,alpha,k_h,k", CASES)
def test_block_form_against_the_oracle(n, X, Y, alpha, k_h, k):
    print(f"case blocks n={n} X={X} Y={Y} alpha={alpha} k_h={k_h} k={k}", flush=True)
    rs = reads_of(n % 977, n, k)
    reads = torch.from_numpy(rs.reads).cuda()
    offs = torch.from_numpy(rs.offsets.view(np.int64)).cuda()
    g = P.run_kmerco(reads, offs, k, 2, X, Y, alpha, k_h)
    c = oracle.run_kmerco(rs.reads, rs.offsets, k, 2, X, Y, alpha, k_h)
    for name, a, b in zip(["words", "distinct", "trust", "err"], g[:4], c[:4]):
        assert np.array_equal(np.asarray(a, dtype=np.uint64), np.asarray(b, dtype=np.uint64)), name
    assert g[4] == c[4]


# (bases, X, Y, alpha, k_h, k, by_records): the buckets of positions that the
# first-seen records are sorted by grow from 2^12 to 2^19 positions with the
# call, and the scan of the tiles' counts takes a second workgroup past 4096
# tiles; the forced winner passes are the path they are compared with as well
MARKS = [
    (2_097_152, 601, 607, 8, 1, 25, False), (2_097_153, 601, 607, 8, 2, 25, False),
    (4_194_304, 601, 607, 8, 1, 25, False), (4_194_305, 601, 607, 8, 1, 25, True),
    (16_777_217, 2707, 2711, 8, 1, 31, False), (16_777_217, 2707, 2711, 8, 1, 31, True),
]


@pytest.mark.parametrize("n,X,Y,alpha,k_h,k,by_records", MARKS)
def test_marks_against_the_oracle(n, X, Y, alpha, k_h, k, by_records, monkeypatch):
    if by_records:
        monkeypatch.setenv("KMERCO_WINNER_RECORDS", "1")
    test_block_form_against_the_oracle(n, X, Y, alpha, k_h, k)


def test_the_largest_marks_match_the_winner_passes(monkeypatch):
    n, k = 67_108_865, 31  # buckets of 2^18 positions
    print(f"case marks n={n}", flush=True)
    rs = reads_of(5, n // 16, k)
    reads = torch.from_numpy(np.tile(rs.reads, 17)[:n].copy()).cuda()
    offs = torch.tensor([0, n // 3, n // 3 + 40, n], dtype=torch.int64).cuda()
    out = []
    for forced in (False, True):
        if forced:
            monkeypatch.setenv("KMERCO_WINNER_RECORDS", "1")
        out.append([np.asarray(a) for a in P.run_kmerco(reads, offs, k, 2, 2707, 2711, 8, 1)[:4]])
    for a, b in zip(*out):
        assert np.array_equal(a, b)


# (bases, bases of one repeated k-mer at their start): the second level holds a
# superblock's entries of a bucket in registers and LDS unless one wavefront's
# runs, or the bucket, hold more than that
@pytest.mark.parametrize("n,hot", [(300_000, 1_000), (300_000, 5_000), (600_000, 60_000)])
def test_uneven_buckets_against_the_oracle(n, hot):
    print(f"case uneven n={n} hot={hot}", flush=True)
    rs = reads_of(3, n, 31)
    rs.reads[:hot] = ord("A")
    reads = torch.from_numpy(rs.reads).cuda()
    offs = torch.from_numpy(rs.offsets.view(np.int64)).cuda()
    g = P.run_kmerco(reads, offs, 31, 2, 3833, 3837, 8, 1)
    c = oracle.run_kmerco(rs.reads, rs.offsets, 31, 2, 3833, 3837, 8, 1)
    for name, a, b in zip(["words", "distinct", "trust", "err"], g[:4], c[:4]):
        assert np.array_equal(np.asarray(a, dtype=np.uint64), np.asarray(b, dtype=np.uint64)), name
    assert g[4] == c[4]


# (bases, X, Y, alpha, k_h, k): regions of few entries, which are worked by
# entry: one and two cells a thread, positions that hit a counter twice,
# saturating counters, a last region past the countBF's end
@pytest.mark.parametrize("n,X,Y,alpha,k_h,k", [
    (400_000, 3833, 3837, 8, 1, 55), (400_000, 3833, 3837, 8, 3, 25),
    (400_000, 3833, 3837, 5, 2, 31), (400_000, 3833, 3837, 4, 8, 31),
    (400_000, 3833, 3837, 16, 1, 31),  # its cells do not fit: by counter
    (30_000, 5779, 5813, 8, 1, 31),    # 16404 regions: partitioned plan
])
def test_sparse_regions_against_the_oracle(n, X, Y, alpha, k_h, k):
    test_block_form_against_the_oracle(n, X, Y, alpha, k_h, k)


# the same regions with their records in room of their own: forced winner
# records, and several chunks whose records wait for the last one's counters
@pytest.mark.parametrize("n,hot,alpha,k_h,chunk", [
    (400_000, 0, 8, 1, None), (400_000, 0, 5, 3, None), (400_000, 30_000, 4, 1, None),
    (400_000, 0, 8, 1, 1 << 17), (400_000, 30_000, 4, 1, 1 << 17),
])
def test_sparse_regions_with_own_records(n, hot, alpha, k_h, chunk, monkeypatch):
    print(f"case own records n={n} hot={hot} alpha={alpha} k_h={k_h} chunk={chunk}", flush=True)
    monkeypatch.setenv("KMERCO_WINNER_RECORDS", "1")
    if chunk:
        monkeypatch.setenv("KMERCO_CHUNK_POSITIONS", str(chunk))
    rs = reads_of(7, n, 31)
    rs.reads[:hot] = ord("A")
    reads = torch.from_numpy(rs.reads).cuda()
    offs = torch.from_numpy(rs.offsets.view(np.int64)).cuda()
    g = P.run_kmerco(reads, offs, 31, 2, 5779, 5813, alpha, k_h)
    c = oracle.run_kmerco(rs.reads, rs.offsets, 31, 2, 5779, 5813, alpha, k_h)
    for name, a, b in zip(["words", "distinct", "trust", "err"], g[:4], c[:4]):
        assert np.array_equal(np.asarray(a, dtype=np.uint64), np.asarray(b, dtype=np.uint64)), name
    assert g[4] == c[4]


# Several hash functions leave up to k_h first-seen records a position: novel
# reads over more than two of the winner passes' blocks of 2^19 positions, one-
# and two-level lists, regions worked by counter and by entry
@pytest.mark.parametrize("k_h,X,Y", [(2, 1009, 1013), (3, 1009, 1013), (8, 1009, 1013),
                                     (2, 5779, 5813), (3, 5779, 5813)])
def test_winner_records_of_several_hash_functions(k_h, X, Y, monkeypatch):
    monkeypatch.setenv("KMERCO_WINNER_RECORDS", "1")
    n, k = 3 * (1 << 19) + 12_345, 31
    print(f"case records of several hash functions k_h={k_h} X={X} Y={Y}", flush=True)
    rs = synth.random_reads(11 + k_h, n // 1000, 1000, 1000, k=k, p_n=0.0001)
    reads = torch.from_numpy(rs.reads).cuda()
    offs = torch.from_numpy(rs.offsets.view(np.int64)).cuda()
    g = P.run_kmerco(reads, offs, k, 2, X, Y, 8, k_h)
    c = oracle.run_kmerco(rs.reads, rs.offsets, k, 2, X, Y, 8, k_h)
    for name, a, b in zip(["words", "distinct", "trust", "err"], g[:4], c[:4]):
        assert np.array_equal(np.asarray(a, dtype=np.uint64), np.asarray(b, dtype=np.uint64)), name
    assert g[4] == c[4]


def test_winner_records_past_the_first_bucket(monkeypatch):
    """More records than positions in a whole bucket of 2^24 positions, against the form that
    sorts its records in the region pass."""
    n, k = (1 << 24) + (1 << 21) + 777, 31
    print(f"case records of two hash functions n={n}", flush=True)
    rs = synth.random_reads(23, n // 1000, 1000, 1000, k=k)
    reads = torch.from_numpy(rs.reads).cuda()
    offs = torch.from_numpy(rs.offsets.view(np.int64)).cuda()
    out = []
    for forced in (False, True):
        if forced:
            monkeypatch.setenv("KMERCO_WINNER_RECORDS", "1")
        out.append(P.run_kmerco(reads, offs, k, 2, 2707, 2711, 8, 2))
    for a, b in zip(out[0][:4], out[1][:4]):
        assert np.array_equal(np.asarray(a), np.asarray(b))
    assert out[0][4] == out[1][4]


@pytest.mark.parametrize("k_h", [1, 2])
def test_a_chunk_beyond_the_sorted_records(k_h, monkeypatch):
    """One chunk above 2^28 positions, which takes the winner passes unforced, against the same
    insert with them turned off (two chunks, whose records the region pass sorts)."""
    n, k = (1 << 28) + (1 << 20) + 4321, 31
    print(f"case large chunk k_h={k_h} n={n}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(17)
    letters = torch.tensor(list(b"ACGT"), dtype=torch.uint8, device="cuda")
    reads = torch.empty(n, dtype=torch.uint8, device="cuda")
    for a in range(0, n, 1 << 26):
        m = min(1 << 26, n - a)
        reads[a:a + m] = letters[torch.randint(0, 4, (m,), generator=g, device="cuda")]
    offs = torch.tensor([0, n // 3, n // 3 + 40, n], dtype=torch.int64, device="cuda")
    out = []
    for chunks in (1, 2):
        if chunks == 2:
            monkeypatch.setenv("KMERCO_WINNER_RECORDS", "0")
        bf = P.CountBF(5779, 5813, 8, k_h)
        assert bf.plan(n)["n_chunks"] == chunks
        d, t, nt, e, ne = bf.insert_classify(reads, offs, k, 2)
        bf.sync()
        nd, nt, ne = int(bf.n_distinct.item()), int(nt.item()), int(ne.item())
        out.append([bf.words.clone(), d[:nd].clone(), t[:nt].clone(), e[:ne].clone()])
        bf.close()
        del d, t, e
    for name, a, b in zip(["words", "distinct", "trust", "err"], *out):
        assert torch.equal(a, b), name


def test_more_superblocks_than_threads():
    """A region pass of more than 1024 superblocks takes their runs in turns: five regions in
    partitions of four, whose superblocks are single blocks of 2^15 positions."""
    n, k = 40_000_001, 31
    print(f"case many superblocks n={n}", flush=True)
    rs = reads_of(29, n // 8, k)
    reads = torch.from_numpy(np.tile(rs.reads, 9)[:n].copy()).cuda()
    offs = torch.tensor([0, n // 3, n // 3 + 40, n], dtype=torch.int64).cuda()
    out = []
    for env in ({"KMERCO_PART_LOG": "2"}, {"KMERCO_PATH": "direct"}):
        with pytest.MonkeyPatch.context() as m:
            for name, v in env.items():
                m.setenv(name, v)
            bf = P.CountBF(101, 101, 8, 1)
            plan = bf.plan(n)
            bf.close()
            assert plan["path"] == ("direct" if out else "partitioned")
            assert out or plan["n_regions"] == 5
            out.append(P.run_kmerco(reads, offs, k, 2, 101, 101, 8, 1))
    for name, a, b in zip(["words", "distinct", "trust", "err"], out[0][:4], out[1][:4]):
        assert np.array_equal(np.asarray(a), np.asarray(b)), name
    assert out[0][4] == out[1][4]


def check_hot(n, hot, X, Y, k_h, what):
    print(f"case {what} n={n} hot={hot} k_h={k_h}", flush=True)
    rs = reads_of(31, n, 31)
    rs.reads[n // 3:n // 3 + hot] = ord("A")
    reads = torch.from_numpy(rs.reads).cuda()
    offs = torch.from_numpy(rs.offsets.view(np.int64)).cuda()
    g = P.run_kmerco(reads, offs, 31, 2, X, Y, 8, k_h)
    c = oracle.run_kmerco(rs.reads, rs.offsets, 31, 2, X, Y, 8, k_h)
    for name, a, b in zip(["words", "distinct", "trust", "err"], g[:4], c[:4]):
        assert np.array_equal(np.asarray(a, dtype=np.uint64), np.asarray(b, dtype=np.uint64)), name
    assert g[4] == c[4]


# Up to eight superblocks share the region pass's 16 wavefronts: five regions,
# superblocks of 13 blocks of 4096 positions, so many of them and a tail
@pytest.mark.parametrize("supers", [1, 2, 3, 4, 5, 8, 9, 16, 17])
@pytest.mark.parametrize("hot", [0, 30_000])
def test_wavefronts_share_a_superblock(supers, hot, monkeypatch):
    monkeypatch.setenv("KMERCO_PART_LOG", "2")
    check_hot(13 * 4096 * supers - 1234, hot, 101, 101, 1, f"{supers} superblocks")


# The same for regions worked by entry (superblocks of 2.75 M positions), with
# regions and buckets of more entries than are held, mostly of one counter
@pytest.mark.parametrize("n,hot,k_h", [(300_000, 250_000, 1), (300_000, 250_000, 3),
                                       (3_000_000, 1_000_000, 1), (6_000_000, 300_000, 1)])
def test_wavefronts_share_a_superblock_by_entry(n, hot, k_h):
    check_hot(n, hot, 5779, 5813, k_h, "by entry")


def check_novel(n, X, Y, k_h, what):
    print(f"case {what} n={n} k_h={k_h}", flush=True)
    rs = synth.random_reads(37 + k_h, 1, n, n, k=31)
    reads = torch.from_numpy(rs.reads).cuda()
    offs = torch.from_numpy(rs.offsets.view(np.int64)).cuda()
    g = P.run_kmerco(reads, offs, 31, 2, X, Y, 8, k_h)
    c = oracle.run_kmerco(rs.reads, rs.offsets, 31, 2, X, Y, 8, k_h)
    for name, a, b in zip(["words", "distinct", "trust", "err"], g[:4], c[:4]):
        assert np.array_equal(np.asarray(a, dtype=np.uint64), np.asarray(b, dtype=np.uint64)), name
    assert g[4] == c[4]


# Regions of about 120 new k-mers, whose records wait in LDS: some have more
# than wait there, and a workgroup's regions fill the room several times; then
# the first averages past it
@pytest.mark.parametrize("n", [2_000_000, 2_099_742, 2_200_000])
def test_records_of_few_entries(n):
    check_novel(n, 5779, 5813, 1, "records of few entries")


# New k-mers beyond the entries that are held: a few a region, and (nearly all
# entries in the first of two regions) more than their room
@pytest.mark.parametrize("n,X,Y,k_h,part_log", [(40_900, 101, 101, 1, "2"), (20_450, 101, 101, 2, "2"),
                                                (16_400, 1, 2053, 1, "0"), (8_200, 1, 2053, 2, "0")])
def test_records_beyond_the_held_entries(n, X, Y, k_h, part_log, monkeypatch):
    monkeypatch.setenv("KMERCO_PART_LOG", part_log)
    check_novel(n, X, Y, k_h, "records beyond the held entries")
    monkeypatch.setenv("KMERCO_WINNER_RECORDS", "1")
    check_novel(n, X, Y, k_h, "own records beyond the held entries")


# Regions worked by entry whose cells are not 1024 or 2048: 256 and 512 cells,
# and 4096 and 8192 that stay in memory, flat and own records, a counter hit
# twice by a position, saturating ones, more entries than are held
@pytest.mark.parametrize("alpha,k_h,n,X,Y,part_log", [
    (1, 1, 400_000, 1511, 1523, None),    # 8990 regions of 256 cells
    (1, 3, 200_000, 1511, 1523, None),
    (2, 2, 400_000, 2003, 2011, None),    # 7868 regions of 512 cells
    (3, 8, 60_000, 2003, 2011, None),
    (16, 1, 400_000, 5779, 5813, None),   # 8202 regions of 4096 cells
    (16, 2, 400_000, 5779, 5813, None),
    (32, 1, 400_000, 1009, 1013, "2"),    # 125 regions of 8192 cells
    (20, 3, 130_000, 1009, 1013, "2"),
    (32, 1, 32_760, 89, 719, "2"),        # 8 regions of 4095 entries on average
])
@pytest.mark.parametrize("own", [False, True])
def test_sparse_regions_of_other_cells(alpha, k_h, n, X, Y, part_log, own, monkeypatch):
    if part_log:
        monkeypatch.setenv("KMERCO_PART_LOG", part_log)
    if own:
        monkeypatch.setenv("KMERCO_WINNER_RECORDS", "1")
    test_block_form_against_the_oracle(n, X, Y, alpha, k_h, 31)


@pytest.mark.parametrize("alpha,X,Y", [(1, 1511, 1523), (16, 5779, 5813)])
def test_sparse_regions_of_other_cells_overfull(alpha, X, Y):
    """Most entries in one region, over counters that are not zero before."""
    n = 400_000
    print(f"case other cells, overfull alpha={alpha}", flush=True)
    rs = reads_of(41, n, 31)
    rs.reads[1000:300_000] = ord("A")
    twice = synth.concat_reads([rs, rs])
    one = [torch.from_numpy(a).cuda() for a in (rs.reads, rs.offsets.view(np.int64))]
    bf = P.CountBF(X, Y, alpha, 1)
    lists = []
    for _ in range(2):
        d, t, nt, e, ne = bf.insert_classify(*one, 31, 1)
        bf.sync()
        lists.append((d[:int(bf.n_distinct.item())].clone(), t[:int(nt.item())].clone()))
    c = oracle.run_kmerco(twice.reads, twice.offsets, 31, 1, X, Y, alpha, 1)
    assert np.array_equal(bf.words.cpu().numpy().view(np.uint64), np.asarray(c[0], dtype=np.uint64))
    assert np.array_equal(lists[0][0].cpu().numpy().view(np.uint64), np.asarray(c[1], dtype=np.uint64))
    assert lists[1][1].numel() == 0
    bf.close()


# Sparse regions of a countBF small enough for the one-level form: the line
# between the forms in regions (1535 | 1536) and in entries, from a few bases
# on, chunks of which the last is sparser than the others
@pytest.mark.parametrize("n,X,Y,alpha,k_h,chunk", [
    (500, 1811, 1737, 8, 1, None),        # 1536 regions
    (40_000, 1811, 1735, 8, 1, None),     # 1535
    (40_000, 1811, 1737, 8, 3, None),
    (3_145_728, 1811, 1737, 8, 1, None), (3_145_729, 1811, 1737, 8, 1, None),  # 2048 a region
    (300_000, 2707, 2711, 16, 1, None),   # 1792 regions of 4096 cells
    (300_000, 1009, 1013, 2, 2, None),    # 1997 regions of 512 cells
    (4_000_000, 1811, 1737, 8, 1, 3_300_000 // 1024 * 1024),
])
def test_sparse_regions_of_smaller_countbfs(n, X, Y, alpha, k_h, chunk, monkeypatch):
    if chunk:
        monkeypatch.setenv("KMERCO_CHUNK_POSITIONS", str(chunk))
    test_block_form_against_the_oracle(n, X, Y, alpha, k_h, 31)


# Regions of 8192 counters worked by entry: from the one-level and the
# partitioned plan, own records, carried chunks, cells in memory
@pytest.mark.parametrize("n,X,Y,alpha,k_h,env", [
    (400_000, 1811, 1741, 8, 1, {}),      # 3080 regions
    (400_000, 1811, 1733, 8, 1, {}),      # 3065: one-level
    (400_000, 4201, 4211, 8, 2, {}),      # 17277: partitioned
    (400_000, 4201, 4211, 8, 1, {"KMERCO_WINNER_RECORDS": "1"}),
    (400_000, 4201, 4211, 8, 1, {"KMERCO_CHUNK_POSITIONS": "131072"}),
    (300_000, 4201, 4211, 16, 1, {}),     # 8639 of 2048 cells
    (300_000, 5779, 5813, 32, 3, {}),     # 8202 of 4096 cells
    (300_000, 1009, 1013, 1, 1, {}),      # 7985 of 128 cells
])
def test_small_sparse_regions(n, X, Y, alpha, k_h, env, monkeypatch):
    monkeypatch.setenv("KMERCO_REGION_COUNTERS", "8192")
    for name, v in env.items():
        monkeypatch.setenv(name, v)
    test_block_form_against_the_oracle(n, X, Y, alpha, k_h, 31)


# Carried chunks of which the last is worked by entry (its own records in the
# regions' room, unforced), after denser ones and sparse ones
@pytest.mark.parametrize("n,chunk,X,Y,alpha", [
    (400_000, 1 << 17, 5779, 5813, 8), (400_000, 1 << 17, 3833, 3837, 4),
    (300_500, 300_032, 1511, 1523, 1), (4_000_000, 3_999_744, 1811, 1737, 8),
])
def test_carried_chunks_by_entry(n, chunk, X, Y, alpha, monkeypatch):
    monkeypatch.setenv("KMERCO_CHUNK_POSITIONS", str(chunk))
    test_block_form_against_the_oracle(n, X, Y, alpha, 1, 31)
