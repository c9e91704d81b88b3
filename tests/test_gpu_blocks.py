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
    (500_000, 3833, 3837, 8, 1, 31),          # 7182 regions: counted binning
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
