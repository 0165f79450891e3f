"""CPU checks of the draw kernels' launch arithmetic (csrc/launch_shape.h, plain C++): compiled here with the host compiler
and gone through for every size, since a wrong share or a load past a row shows in no result that a small launch gives."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1409_5402_amd", "csrc")

SHIM = r"""
#include "launch_shape.h"
#include <vector>
using namespace same;

// Positions of a launch that are not drawn exactly once when every group that has a workgroup takes tickets until none is left.
static long undrawn(long n, long resident)
{
    std::vector<unsigned char> drawn(n, 0);
    long wrong = 0;
    auto draw = [&](long from, long size) {
        for (long i = from; i < from + size && i < n; ++i) if (drawn[i]++) ++wrong;
    };
    const Shares s = shares_for(n, resident);
    bool has[kGroups] = {};
    for (long b = 0; b < s.waves; ++b) { draw(b * s.first, s.first); has[ticket_group((uint32_t)b)] = true; }
    if ((long)s.waves * s.first < n)
        for (uint32_t g = 0; g < kGroups; ++g)
            for (uint32_t t = 0; has[g]; ++t) {
                const Share h = share_of_ticket(t, g, (uint32_t)s.waves, s.first, n);
                if (h.from >= n) break;
                draw(h.from, h.size);
            }
    for (long i = 0; i < n; ++i) if (!drawn[i]) ++wrong;
    return wrong;
}
// A launch in which every workgroup wants more chunks than its own share, `busy` of them in their turn: batches that start
// inside a part of the pool which has been handed out before.
static long owners_of_one_chunk(unsigned waves, unsigned share, unsigned chunks, unsigned busy)
{
    long wrong = 0;
    uint32_t counter = 0;
    uint32_t handed = waves * share;
    for (unsigned w = 0; w < waves; ++w)
        for (unsigned turn = 0; turn < busy; ++turn) {
            const Chunks c = chunk_batch(counter, waves, share, chunks);
            counter += 1u;
            if (c.next == c.end) break;                            // dry: asks no more
            if (c.next != handed || c.end > chunks) ++wrong;
            handed = c.end;
        }
    return wrong + (handed != chunks);
}
extern "C" {
int t_block_len(int K) { return block_len(K); }
int t_blocks_in_use(int K) { return blocks_in_use(K); }
int t_blocks_fill_row(int K) { return blocks_fill_row(K); }
long t_undrawn(long n, long workgroups) { return undrawn(n, whole_groups(workgroups)); }
long t_owners_of_one_chunk(unsigned waves, unsigned share, unsigned chunks, unsigned busy) { return owners_of_one_chunk(waves, share, chunks, busy); }
int t_lds_groups(long bytes) { return lds_groups(bytes); }
// Numbers of topics for which the rule and the forms of the kernel that exist contradict each other, or whose form has no such row.
long t_theta_rows_wrong()
{
    long wrong = 0;
    for (int K = 1; K <= 2048; ++K) {
        const int quads = block_len(K) / 4;
        const bool on = theta_rows(K), one_batch = quads <= 7, one_row = K > 128 && K <= 1024;
        wrong += on && !(one_batch && one_row && theta_rows_some(quads));
        wrong += theta_rows_all(quads, K % 4 == 0) && !on;
    }
    return wrong;
}
// Counts of a D x K matrix that the workgroups of the totals do not take exactly once, accesses off a 16-byte boundary, and workgroups
// with less than half of their threads in use where there are several turns.
long t_totals_counts_wrong(unsigned D, int K)
{
    const TotalsSplit s = totals_split(K);
    const TotalsBlocks t = totals_blocks(s, D);
    std::vector<unsigned char> taken((size_t)D * K, 0);
    const size_t row = 4 * (size_t)s.units;
    long wrong = row != (size_t)s.fold * K || s.per * s.groups > 256 || s.per * s.turns < s.units || (s.turns > 1 && 2 * s.per * s.groups < 256);
    for (unsigned block = 0; block < t.blocks; ++block) {
        const Rows b = rows_of_block(block / s.turns, t.rows_per_block, t.rows);
        for (unsigned i = 0; i < 256; ++i) {
            const unsigned group = i / s.per;
            const int unit = (int)(block % s.turns) * s.per + (int)(i % s.per);
            if (group >= (unsigned)s.groups || unit >= s.units) continue;
            for (unsigned r = b.from + group; r < b.to; r += s.groups)
                for (int c = 0; c < 4; ++c) {
                    const size_t at = r * row + 4 * unit + c;
                    if (at >= taken.size() || taken[at]++ || (at - c) % 4 != 0 || at % K != (size_t)((4 * unit + c) % K)) ++wrong;
                }
        }
        if (block == 0) for (size_t i = t.rows * row; i < taken.size(); ++i) if (taken[i]++) ++wrong;
    }
    for (unsigned char c : taken) if (!c) ++wrong;
    return wrong;
}
long t_totals_blocks(unsigned D, int K) { return totals_blocks(totals_split(K), D).blocks; }
int t_theta_rows(int K) { return theta_rows(K); }
int t_groups_per_unit(int K, int most) { return groups_per_unit(K, most); }
// Rows near `rows` that belong to no workgroup, to two, or to one past the end.
long t_rows_without_owner(unsigned rows, unsigned per_block)
{
    const uint32_t blocks = blocks_of_rows(rows, per_block);
    long wrong = rows_of_block(blocks - 1, per_block, rows).to != rows;
    for (uint32_t b = blocks > 5 ? blocks - 5 : 0; b < blocks; ++b) {
        const Rows r = rows_of_block(b, per_block, rows);
        wrong += r.from >= r.to || r.to > rows || (b > 0 && rows_of_block(b - 1, per_block, rows).to != r.from);
    }
    return wrong;
}
// Documents of one thread's loop that are not in [0, D) or do not ascend; the last one must be within a stride of D.
long t_documents_out_of_range(int first, int step, int D)
{
    long wrong = 0;
    int32_t d = first, before = first - 1;
    if (d < D) do { wrong += d < 0 || d >= D || d <= before; before = d; } while (wrong == 0 && next_document(d, step, D));
    return wrong + (first < D && D - step > before);
}
// The totals' memory: copies that 16-byte stores cannot clear whole, arrays that overlap or end behind it.
int t_totals_wrong(int K)
{
    const TotalsLayout t = totals_layout(K);
    const size_t ends[2] = {t.copies + t.copy_words, t.totals + (size_t)K};
    int wrong = 8 * t.copies % 16 != 0 || t.copy_words != (size_t)nk_copies_for(K) * K;
    wrong += !(ends[0] <= t.totals || ends[1] <= t.copies) || ends[0] > t.words || ends[1] > t.words;
    return wrong;
}
// Nonzeros that the last turns of the E-step's loop over a document of n name, rounds loaded ahead included, outside [0, n).
long t_nonzeros_out_of_range(unsigned n, unsigned round)
{
    long wrong = 0;
    const unsigned last = (n - 1u) / (2u * round);
    for (unsigned t = last > 3u ? last - 3u : 0u; t <= last; ++t)
        for (unsigned at = 0; at < 3u * round; ++at) {
            const long i = (long)t * 2 * round + at, got = vb_nonzero(t * 2u * round, at, n);
            wrong += got != (i < (long)n ? i : (long)n - 1) || at >= kVbAhead;
        }
    return wrong;
}
unsigned t_chunk_share(unsigned chunks, long n, long waves) { return chunk_share(chunks, n, waves); }
int t_scan_first_topic(int hl, int T, int nblk) { return scan_first_topic(hl, T, nblk); }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    where = tmp_path_factory.mktemp("launch_shape")
    src, so = where / "shim.cpp", where / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-I", CSRC,
                    str(src), "-o", str(so)], check=True)
    so = ctypes.CDLL(str(so))
    so.t_chunk_share.argtypes = [ctypes.c_uint, ctypes.c_long, ctypes.c_long]
    so.t_chunk_share.restype = ctypes.c_uint
    so.t_lds_groups.argtypes = [ctypes.c_long]
    so.t_undrawn.argtypes = [ctypes.c_long] * 2
    so.t_undrawn.restype = ctypes.c_long
    so.t_rows_without_owner.argtypes = [ctypes.c_uint] * 2
    so.t_rows_without_owner.restype = ctypes.c_long
    so.t_documents_out_of_range.restype = ctypes.c_long
    so.t_nonzeros_out_of_range.argtypes = [ctypes.c_uint] * 2
    so.t_nonzeros_out_of_range.restype = ctypes.c_long
    so.t_owners_of_one_chunk.argtypes = [ctypes.c_uint] * 4
    so.t_owners_of_one_chunk.restype = ctypes.c_long
    return so


def test_scan_stays_inside_the_row(lib):
    """Loads without bounds: every lane's block lies inside the row for every number of topics that takes them, and the
    blocks in use are each some lane's."""
    unguarded = 0
    for K in range(4, 2049, 4):
        if not lib.t_blocks_fill_row(K):
            continue
        unguarded += 1
        T, nblk = lib.t_block_len(K), lib.t_blocks_in_use(K)
        first = [lib.t_scan_first_topic(hl, T, nblk) for hl in range(32)]
        assert max(first) + T <= K, (K, T, nblk)
        assert first[:nblk] == [T * l for l in range(nblk)], K
    assert unguarded > 100


@pytest.mark.parametrize("workgroups", [1, 32, 100, 224, 255, 256, 384, 1000, 3072, 4096, 5120])
def test_every_position_has_one_share(lib, workgroups):
    """Whatever number of workgroups a device holds at once: the static shares and the halving ones
    cover every launch position once, and no ticket group is without a workgroup that draws its shares."""
    for n in (1, 63, 64, 65, 128 * 256, 128 * 256 + 1, 128 * workgroups, 128 * workgroups + 1, 1000 * workgroups + 77, 2500 * workgroups + 1, 3_000_017):
        assert lib.t_undrawn(n, workgroups) == 0, n


@pytest.mark.parametrize("waves,chunks", [(1, 300), (4096, 100_000), (1 << 20, 50_000_000), ((1 << 24) + 9, 1000), ((1 << 25) - 1, (1 << 31) - 1)])
def test_a_chunk_has_one_owner(lib, waves, chunks):
    """Workgroups that find the pool used up still add to its counter: up to the 2^25 workgroups of the largest launch of the
    Poisson form no batch is handed out twice."""
    share = lib.t_chunk_share(chunks, 64 * waves, waves)
    assert share * waves <= chunks // 2
    assert lib.t_owners_of_one_chunk(waves, share, chunks, 3 if waves > 100 else 1000) == 0


def test_workgroups_per_compute_unit(lib):
    """All that fit up to 1024 topics, then as many as have room for a row of theta each in 32 KB; never none, never more than
    fit."""
    assert [lib.t_groups_per_unit(K, 16) for K in (1, 256, 512, 1024, 1025, 1170, 1171, 1366, 1639, 2048)] == [16, 16, 16, 16, 7, 7, 6, 5, 4, 4]
    assert all(1 <= lib.t_groups_per_unit(K, most) <= most for K in range(1, 2049) for most in (1, 3, 12))


def test_workgroups_that_lds_holds(lib):
    """What a probe measured: launches of one workgroup more per compute unit take twice the time."""
    measured = {8960: 18, 8961: 16, 9472: 16, 10240: 16, 10241: 14, 10496: 14, 11520: 14, 11521: 12, 12544: 12, 12800: 12, 12801: 11}
    assert {lds: lib.t_lds_groups(lds) for lds in measured} == measured


def test_own_chunks_stay_close_together(lib):
    """The workgroups' own shares of the pool follow what a launch needs and not the size of the pool (eight chunks per task
    and more): the chunks in use stay within a few times their number."""
    for n, waves in ((100_000, 1563), (6_000_000, 4096), (60_000_000, 3584), (60_000_000, 937_500)):
        share = lib.t_chunk_share(min(10 * n, 2**31 - 1), n, waves)
        assert share * waves <= n // 2 and share >= n // 2 // waves
        assert lib.t_chunk_share(7, n, waves) == 0 and lib.t_chunk_share(0, n, waves) == 0


def test_topic_totals_have_their_place(lib):
    """The copies of the totals start where a 16-byte store may, whatever the number of topics, and share nothing with the totals."""
    assert [K for K in range(1, 2049) if lib.t_totals_wrong(K)] == []


@pytest.mark.parametrize("round_", [4, 8, 16])
def test_nonzeros_of_a_round_exist(lib, round_):
    """The E-step's rounds, the ones loaded ahead among them, name nonzeros of their document, up to a document of 2^31 - 1."""
    for n in (1, 2, 3, round_, 2 * round_ + 1, 1000, 2**31 - 100, 2**31 - 33, 2**31 - 2, 2**31 - 1):
        assert lib.t_nonzeros_out_of_range(n, round_) == 0, n


def test_lds_arrays_are_aligned_for_the_widest_access():
    """Dynamic LDS that is accessed 16 bytes at a time is declared with that alignment (the E-step's arrays of double are not:
    8 bytes at most)."""
    arrays = []
    for name in sorted(os.listdir(CSRC)):
        with open(os.path.join(CSRC, name)) as f:
            arrays += [(name, line.strip()) for line in f if "extern __shared__" in line]
    assert len(arrays) >= 5
    for name, line in arrays:
        assert "extern __shared__ double" in line or "__align__(16)" in line, (name, line)


def test_theta_rows_only_where_the_kernel_has_them(lib):
    """The rule asks for rows of theta in LDS only at sizes whose form of the draw kernel is instantiated with them (blocks of one
    batch of loads, one row of counts), and at every size where it is instantiated with them alone."""
    assert lib.t_theta_rows_wrong() == 0
    for K, on in ((287, 0), (288, 1), (292, 0), (289, 1), (448, 1), (500, 0), (512, 1), (516, 1), (701, 1), (895, 1), (896, 1), (897, 0), (1024, 0)):
        assert bool(lib.t_theta_rows(K)) == bool(on), K


def test_totals_take_every_count_once(lib):
    """n_dk in rows of one, two or four documents: every count once, on 16-byte boundaries, its topic the thread's own."""
    for D in (1, 2, 3, 4, 7):
        assert [K for K in range(1, 2049) if lib.t_totals_counts_wrong(D, K)] == [], D
    for K in (1, 2, 3, 4, 5, 50, 64, 129, 255, 256, 257, 258, 333, 512, 513, 1001, 1024, 1025, 1030, 2046, 2047, 2048):
        assert lib.t_totals_counts_wrong(2999, K) == 0, K
        assert lib.t_totals_blocks(0, K) == 0 and lib.t_totals_blocks(2**31 - 1, K) <= 1024


def test_registers_left_beside_a_sweep():
    """Four waves of a draw on a SIMD leave registers for the staging of the next minibatch, whose uploads and passes otherwise
    wait for the draw to end.  The numbers are the compiler's, in the metadata of the library built here."""
    msgpack = pytest.importorskip("msgpack")
    from paper_1409_5402_amd import build
    if not os.path.exists(build.LIB):
        build.build()
    with open(build.LIB, "rb") as f:
        image = f.read()
    at = image.index(b"amdhsa.kernels") - 2                        # a map of a few entries, the first key's length before it
    unpacker = msgpack.Unpacker(raw=False, strict_map_key=False)
    unpacker.feed(image[at:at + (4 << 20)])
    registers = {k[".name"]: k[".vgpr_count"] for k in unpacker.unpack()["amdhsa.kernels"]}

    def draw(aligned, quads, theta):
        return registers["_ZN4same11draw_kernelILb0ELb%dELb0ELi%dELb1ELi0ELb0ELb%dEEEvNS_8DrawArgsE" % (aligned, quads, theta)]
    for aligned in (0, 1):
        assert draw(aligned, 1, 0) <= 112
        assert draw(aligned, 2, 0) <= 120
    for theta in (0, 1):
        assert draw(1, 3, theta) <= 120
    assert next(v for k, v in registers.items() if "wl_scan_docs" in k) <= 512 - 4 * 120
