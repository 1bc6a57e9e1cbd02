"""The hand-placed waits and barriers of the windowed block kernel, checked without a GPU.

The statements of the waves that load, shift tile words and store are cut from the kernel's source and compiled for the
host with the accesses replaced by lines of a trace; the matrix-core waves' side of the protocol is written out below.
Two waves may touch the same part of LDS only with a barrier between (a load is in flight from its issue to the wait that
covers it), and every read has to find the chunk or round that it is for."""
import collections
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = os.path.join(ROOT, "paper_2407_12075_amd", "csrc", "tbn_linear_block.hip")

HARNESS = r"""
#include <cstdint>
#include <cstdio>
#include <cstdlib>
static const int32_t n_rounds = N_ROUNDS;
static const uint32_t n_blocks = N_BLOCKS;
static struct { uint32_t x; } gridDim = {1};
constexpr bool WIN = true;
constexpr int NQ = WAVES_LOAD == 2 ? 2 : 1, kOdd = 8 * NQ, kEven = 9 * NQ;
static int vmcnt_imm(int n) { return n; }
static void __builtin_amdgcn_s_waitcnt(int n) { std::printf("vm %d 0\n", n); }
#define __builtin_amdgcn_s_barrier() std::printf("barrier 0 0\n")
template <int N> static void lds_wait() { static_assert(N == 0, ""); std::printf("lds 0 0\n"); }
static void set_block(uint32_t b) { std::printf("block %u 0\n", b); }
static void start_tile() { std::printf("start 0 0\n"); }
static void fetch_tile(int32_t r) { std::printf("fetch %d 0\n", r); }
static void put_tile(int32_t r) { std::printf("put %d 0\n", r); }
static void issue_round_x(int32_t r, int32_t phase) { std::printf("rows %d %d\n", r, phase); }
static void store_unit(int32_t) {}
static void load_wave() {
    uint32_t bid = 0;
    (void)bid;
    @LOAD@
}
static void store_wave() {
    uint32_t bid = 0;
    int32_t m0 = 0, n0 = 0, st_credit = 0, st_total = 0, st_next = 0;
    @STORE@
}
int main(int, char **argv) { if (argv[1][0] == 'l') load_wave(); else store_wave(); }
"""


def _cut(text, begin, end):
    """The text from the one place where `begin` stands up to the next `end`, without `end`."""
    assert text.count(begin) == 1, f"{text.count(begin)} places in {SOURCE} read {begin!r}"
    at = text.index(begin)
    return text[at:text.index(end, at)]


def _statements(persist):
    text = open(SOURCE).read()
    win = _cut(text, "        // The rounds of the loops below, two at a time (even, odd).", "    } else if (wave >= 4) {")
    win = win[win.index("if constexpr (PERSIST) {"):]
    one_block = win.index("} else {\n            start_tile();")
    if not persist:
        return win[one_block + len("} else {"):win.index("return;", one_block) + len("return;")], ""
    load = win[len("if constexpr (PERSIST) {"):one_block]
    store = _cut(text, "        int32_t ph = 0;\n        if constexpr (WIN) {", "            // the same turn-round as in the epilogue")
    return load, store + r"""
            std::printf("take 0 %d\n", ph);
            ph = (ph + n_rounds) & 3;
            (void)cur_m0; (void)cur_n0;
            if (!more) return;
        }"""


def _traces(tmp_path, persist, n_rounds, blocks):
    load, store = _statements(persist)
    src, exe = tmp_path / "waves.cpp", str(tmp_path / "waves")
    src.write_text(HARNESS.replace("@LOAD@", load).replace("@STORE@", store))
    res = subprocess.run(["g++", "-std=c++17", "-O0", "-w", f"-DN_ROUNDS={n_rounds}", f"-DN_BLOCKS={blocks}",
                          f"-DWAVES_LOAD={2 if persist else 4}", str(src), "-o", exe], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    run = lambda kind: [(op, int(a), int(b)) for op, a, b in
                        (l.split() for l in subprocess.run([exe, kind], capture_output=True, text=True, check=True).stdout.splitlines())]
    traces = {}
    for wave in range(4, 8):
        storing = persist and wave >= 6
        quarters = (2 * (wave & 1), 2 * (wave & 1) + 1) if persist else (wave & 3,)
        traces[wave] = (quarters, run("s" if storing else "l"))
    return traces


Access = collections.namedtuple("Access", "region write wave begin end begin_seq end_seq tag")


def _accesses(wave, quarters, trace, n_rounds):
    """What one wave does to LDS: (region, from and to which barrier interval, from and to which step of the wave)."""
    out, flight, writes = [], collections.deque(), []   # loads in flight; LDS writes since the last wait for LDS
    epoch = block = taken = 0
    fetched = put = None
    for seq, (op, a, b) in enumerate(trace):
        if op == "barrier":
            epoch += 1
        elif op == "vm":
            while len(flight) > a:
                region, tag, e, s = flight.popleft()
                out.append(Access(region, True, wave, e, epoch, s, seq, tag))
        elif op == "lds":
            out += [Access(r, True, wave, e, epoch, s, seq, tag) for r, tag, e, s in writes]
            writes = []
        elif op == "block":
            block, fetched, put = a, None, None
        elif op == "start":
            put = None
        elif op == "fetch":
            assert a == (0 if fetched is None else fetched + 2), "chunks are fetched in order: positions advance with the calls"
            fetched = a
            flight += [(("raw", a // 2 % 3, q), (block, a // 2), epoch, seq) for q in quarters]
        elif op == "rows":
            flight += [(("ring", (a + b) % 4, q), (block, a), epoch, seq) for q in quarters for _ in range(8)]
        elif op == "put":
            assert a == (0 if put is None else put + 2), "chunks are put in place in order: positions advance with the calls"
            put = a
            for q in quarters:   # fifth word: first word of the row's next piece
                nxt = a // 2 if q < 2 else a // 2 + 1
                out.append(Access(("raw", a // 2 % 3, q), False, wave, epoch, epoch, seq, seq, (block, a // 2)))
                out.append(Access(("raw", nxt % 3, q ^ 2), False, wave, epoch, epoch, seq, seq, (block, nxt)))
                writes.append((("tile", a // 2 % 3, q), (block, a // 2), epoch, seq))
        elif op == "take":   # blocks are taken in order
            out += [Access(("ring", s, q), False, wave, epoch, epoch, seq, seq, ("sums", taken)) for s in _exchange(n_rounds, b) for q in range(4)]
            taken += 1
    out += [Access(r, True, wave, e, 1 << 30, s, 1 << 30, tag) for r, tag, e, s in flight]
    assert not writes, "LDS writes that no wait covers"
    return out


def _exchange(n_rounds, ph):
    first = (n_rounds - 2 + ph) % 4
    return first, (first + 1) % 4


def _multiplying(li, persist, n_rounds, blocks):
    """Matrix-core wave li: K group li / 2, column half li % 2.  Reads that the last round requests of a round that does not
    exist are left out: nothing uses them."""
    out, seq, epoch, ph = [], 0, 1, 0   # (behind the barrier "the words of the first chunks are there")
    grp, wn = li >> 1, li & 1

    def access(region, write, tag):
        nonlocal seq
        seq += 1
        out.append(Access(region, write, li, epoch, epoch, seq, seq, tag))

    def rows(block, r):
        for q in (2 * grp, 2 * grp + 1):
            access(("ring", (r + ph) % 4, q), False, (block, r))

    def signs(block, r):
        access(("tile", r // 2 % 3, 2 * (r & 1) + wn), False, (block, r // 2))

    for block in range(blocks):
        epoch += 1
        signs(block, 0)
        rows(block, 0)
        for g in range(n_rounds):
            epoch += 1
            rows(block, g)
            if g + 1 < n_rounds:
                signs(block, g + 1)
                rows(block, g + 1)
        epoch += 1
        area = _exchange(n_rounds, ph) if persist else (0, 1)
        part = lambda w: [("ring", area[w >> 1], 2 * (w & 1)), ("ring", area[w >> 1], 2 * (w & 1) + 1)]
        for r in part(li ^ 2):
            access(r, True, ("half", block))
        epoch += 1
        for r in part(li):
            access(r, False, ("half", block))
        if persist:
            for r in part(li):
                access(r, True, ("sums", block))
            epoch += 1
            ph = (ph + n_rounds) % 4
    return out, epoch


def _check(tmp_path, persist, n_rounds, blocks):
    accesses, barriers = [], set()
    for wave, (quarters, trace) in _traces(tmp_path, persist, n_rounds, blocks).items():
        accesses += _accesses(wave, quarters, trace, n_rounds)
        barriers.add(sum(op == "barrier" for op, _, _ in trace))
    for li in range(4):
        acc, n = _multiplying(li, persist, n_rounds, blocks)
        accesses += acc
        barriers.add(n)
    assert len(barriers) == 1, f"the waves pass different numbers of barriers: {barriers}"
    regions = collections.defaultdict(list)
    for a in accesses:
        regions[a.region].append(a)
    faults = []
    for region, acc in regions.items():
        for r in (a for a in acc if not a.write):
            before = None
            for w in (a for a in acc if a.write):
                if w.wave == r.wave:
                    if w.begin_seq <= r.begin_seq <= w.end_seq and w.begin_seq != r.begin_seq:
                        faults.append(f"{region}: wave {r.wave} reads {r.tag} while its own write of {w.tag} is under way")
                    earlier = w.end_seq < r.begin_seq
                else:
                    if w.begin <= r.end and r.begin <= w.end:
                        faults.append(f"{region}: wave {r.wave} reads {r.tag} between the barriers {r.begin} and {r.begin + 1}, "
                                      f"wave {w.wave} writes {w.tag} between {w.begin} and {w.end + 1}")
                    earlier = w.end < r.begin
                if earlier and (before is None or (w.end, w.end_seq) > (before.end, before.end_seq)):
                    before = w
            if before is None or before.tag != r.tag:
                faults.append(f"{region}: wave {r.wave} reads {r.tag} and finds {before and before.tag}")
        writes = [a for a in acc if a.write]
        faults += [f"{region}: waves {v.wave} and {w.wave} write {v.tag} and {w.tag} at the same time"
                   for i, v in enumerate(writes) for w in writes[:i]
                   if (v.begin <= w.end and w.begin <= v.end if v.wave != w.wave else
                       v.begin_seq < w.end_seq and w.begin_seq < v.end_seq and v.tag != w.tag)]
    assert not faults, f"{len(faults)} faults:\n" + "\n".join(sorted(set(faults))[:12])


@pytest.mark.parametrize("n_rounds", [2, 4, 6, 8, 10, 12, 14, 20, 22])
def test_one_block_per_workgroup(tmp_path, n_rounds):
    _check(tmp_path, False, n_rounds, 1)


@pytest.mark.parametrize("n_rounds", [4, 6, 8, 10, 12, 14, 16, 18, 20, 22, 24, 26])
def test_blocks_one_after_the_other(tmp_path, n_rounds):
    _check(tmp_path, True, n_rounds, 4)
