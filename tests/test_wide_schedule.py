"""Schedule of the wide expert GEMM's main loop, on the CPU: its LDS ring is refilled by asynchronous loads
while eight waves read it half a phase apart, with no other order between them than the barriers, the load
counters and the waits.

The main loop's own text (its macros and the driver below them) is compiled for the host with recording
stand-ins for the loads, the fragment reads, the MFMAs, the waits and the barriers.  Every wave's record is
then checked: no load may refill a block of LDS that another wave has not provably finished reading, no read
may run before the block's load has provably landed, and every MFMA must multiply the halves it is meant
to multiply, each stage once."""

import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = os.path.join(ROOT, "paper_2608_24938_amd", "csrc", "k_gemm.hip")

HARNESS = r"""
#include <cstdint>
#include <cstdio>
#include <cstdlib>
typedef uint16_t bf16_t;
static int g_lane;
static char g_lds[160 * 1024];
static const char *reg_base;
struct bf16x8 {
  int id;
  bf16x8 &operator=(const bf16x8 &o) {  // a read: LDS address into a register
    printf("R %ld %ld\n", (long)(reinterpret_cast<const char *>(this) - reg_base),
           (long)(reinterpret_cast<const char *>(&o) - g_lds));
    return *this;
  }
};
struct f32x16 { int id; float &operator[](int) { static float f; return f; } };
static f32x16 model_mfma(const bf16x8 &b, const bf16x8 &a, f32x16 c) {
  printf("M %ld %ld %d\n", (long)(reinterpret_cast<const char *>(&b) - reg_base),
         (long)(reinterpret_cast<const char *>(&a) - reg_base), c.id);
  return c;
}
static void lds_dma16(const bf16_t *g, uint32_t lds) {
  printf("L %ld %u\n", (long)(reinterpret_cast<uintptr_t>(g) / 2), lds);
}
static uint32_t lds_addr(const void *) { return 0; }
static int wide_slot(int r, int q) { return q ^ ((r ^ (r >> 1)) & 7); }
#define ASM(...) printf("A %s\n", #__VA_ARGS__)
#define BUILTIN_NOP(...) (void)0
constexpr int kWideBK = 64, kWideTM = 4, kWideTN = 2;

template <bool DBL, int TMV> static void run(int wave, int lane, int k0, int k1) {
  constexpr int HALF = 128 * kWideBK, NA = DBL ? 1 : 2, NB = DBL ? 4 : 2;
  bf16_t *smem = reinterpret_cast<bf16_t *>(g_lds);
  const int wm = wave >> 2, wn = wave & 3;
  // source of half tile h of A (0 ..) or B (8 ..): column k at h << 20 | k
  const bf16_t *sa[NA][2], *sb[NB][2];
  auto source = [&](int h) { return reinterpret_cast<const bf16_t *>(((uintptr_t)h << 20 | (uintptr_t)(k0 * kWideBK)) * 2); };
  for (int u = 0; u < 2; ++u) {
    for (int h = 0; h < NA; ++h) sa[h][u] = source(h);
    for (int g = 0; g < NB; ++g) sb[g][u] = source(8 + g);
  }
  f32x16 acc[kWideTM][kWideTN];
  for (int i = 0; i < kWideTM; ++i)
    for (int j = 0; j < kWideTN; ++j) acc[i][j].id = i * kWideTN + j;
  struct { bf16x8 fa[2][4], fb[2][4]; } regs;
  reg_base = reinterpret_cast<const char *>(&regs);
  bf16x8 (&fa)[2][4] = regs.fa, (&fb)[2][4] = regs.fb;
@BODY@
}

template <bool DBL> static void pick(int tmv, int wave, int lane, int k0, int k1) {
  switch (tmv) {
    case 0: if constexpr (DBL) run<DBL, 0>(wave, lane, k0, k1); break;
    case 1: if constexpr (DBL) run<DBL, 1>(wave, lane, k0, k1); break;
    case 2: run<DBL, 2>(wave, lane, k0, k1); break;
    case 3: if constexpr (!DBL) run<DBL, 3>(wave, lane, k0, k1); break;
    case 4: if constexpr (!DBL) run<DBL, 4>(wave, lane, k0, k1); break;
  }
}

int main(int argc, char **argv) {  // dbl tmv-of-waves-0-3 tmv-of-waves-4-7 k0 k1
  const int dbl = atoi(argv[1]), k0 = atoi(argv[4]), k1 = atoi(argv[5]);
  for (int wave = 0; wave < 8; ++wave)
    for (int lane = 0; lane < 64; lane += 8) {
      printf("W %d %d\n", wave, lane);
      const int tmv = atoi(argv[wave < 4 ? 2 : 3]);
      dbl ? pick<true>(tmv, wave, lane, k0, k1) : pick<false>(tmv, wave, lane, k0, k1);
    }
}
"""


def _main_loop():
    src = open(SOURCE).read()
    begin = src.index("  const uint32_t lds0 = lds_addr(smem)")
    last = "  if (wave < 4) EXF_P_BARRIER();"
    body = src[begin: src.index(last, begin) + len(last)]
    assert body.count("bf16x8 fa[2][4], fb[2][4];") == 1
    body = body.replace("bf16x8 fa[2][4], fb[2][4];", "")
    body = body.replace("asm volatile", "ASM")
    body = body.replace("__builtin_amdgcn_mfma_f32_32x32x16_bf16", "model_mfma").replace(", 0, 0, 0)", ")")
    return re.sub(r"__builtin_amdgcn_(sched_barrier|s_setprio)", "BUILTIN_NOP", body)


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    gxx = shutil.which("g++")
    assert gxx, "the schedule model is compiled with g++"
    d = tmp_path_factory.mktemp("wide_schedule")
    (d / "m.cpp").write_text(HARNESS.replace("@BODY@", _main_loop()))
    subprocess.run([gxx, "-std=c++17", "-O0", "-w", str(d / "m.cpp"), "-o", str(d / "m")], check=True)
    return str(d / "m")


class _Thread:
    """One lane's record: its loads, reads and MFMAs, each with the barriers passed before it, and for loads
    and reads the barriers passed when they had provably ended."""

    def __init__(self, wave, lane):
        self.wave, self.lane, self.barriers = wave, lane, 0
        self.loads, self.reads, self.products = [], [], []
        self.reg = {}  # register -> the read that filled it

    def event(self, n, kind, args):
        if kind == "L":
            self.loads.append(dict(n=n, src=int(args[0]), block=int(args[1]) // 1024, at=self.barriers, done=None,
                                   done_n=None))
        elif kind == "R":
            r = dict(n=n, block=int(args[1]) // 1024, addr=int(args[1]), at=self.barriers, done=None, done_n=None)
            self.reads.append(r)
            self.reg[int(args[0])] = r
        elif kind == "M":
            for q in args[:2]:  # an MFMA waits for its own operands
                self._end(self.reg[int(q)], n)
            self.products.append((self.reg[int(args[0])], self.reg[int(args[1])], int(args[2])))
        else:
            text = "".join(args).replace('""', "")
            vm = re.search(r"vmcnt\((\d+)\)", text)
            if vm:
                for q in self.loads[: max(0, len(self.loads) - int(vm.group(1)))]:
                    self._end(q, n)
            if "lgkmcnt(0)" in text:
                for q in self.reads:
                    self._end(q, n)
            if "s_barrier" in text:
                self.barriers += 1

    def _end(self, q, n):
        if q["done"] is None:
            q["done"], q["done_n"] = self.barriers, n


def _threads(model, dbl, tmv, k0, k1):
    out = subprocess.run([model, *map(str, (int(dbl), *tmv, k0, k1))], check=True, capture_output=True, text=True)
    threads = []
    for n, line in enumerate(out.stdout.splitlines()):
        kind, *args = line.split()
        if kind == "W":
            threads.append(_Thread(int(args[0]), int(args[1])))
        else:
            threads[-1].event(n, kind, args)
    return threads


def _before(q, tq, r, tr):
    """The end of q (of thread tq) is ordered before the start of r (of tr): in one wave by a wait between
    them, across waves by a barrier that tq's wave reached after q had ended and tr's passed before r."""
    if q["done"] is None:
        return False
    if tq.wave == tr.wave:
        return q["done_n"] - tq.start < r["n"] - tr.start
    return r["at"] > q["done"]


# full tiles with all or some of the last 128 rows' blocks live, tail tiles with no, one or two live blocks
# a wave; two stages (the least), odd and even counts, ranges that do not begin at stage 0
@pytest.mark.parametrize("dbl,tmv", [(False, (4, 4)), (False, (4, 3)), (False, (3, 2)), (True, (2, 2)), (True, (2, 1)),
                                     (True, (1, 0))])
@pytest.mark.parametrize("k0,k1", [(0, 2), (0, 3), (0, 4), (3, 8), (4, 10), (0, 11)])
def test_ring_is_ordered(model, dbl, tmv, k0, k1):
    threads = _threads(model, dbl, tmv, k0, k1)
    assert len({t.barriers for t in threads}) == 1, "every wave meets every barrier"
    # position inside the wave's program: all lanes of a wave run the same one
    for t in threads:
        first = min(q["n"] for q in t.loads)
        t.start = first
    loaders = [t for t in threads if t.lane == 0]
    by_block = {}
    for t in loaders:
        assert all(q["done"] is not None for q in t.loads), "every load has landed at the end"
        for q in t.loads:
            by_block.setdefault(q["block"], []).append((t, q))
    for t in threads:
        for r in t.reads:
            assert r["done"] is not None
            seen = None
            for tl, q in by_block[r["block"]]:
                landed, refill = _before(q, tl, r, t), _before(r, t, q, tl)
                assert landed or refill, (
                    f"wave {t.wave}: read of LDS block {r['block']} after {r['at']} barriers (ended by "
                    f"{r['done']}) and wave {tl.wave}'s load into it after {q['at']} barriers are unordered")
                if landed and (seen is None or q["n"] > seen["n"]):
                    seen = q
            assert seen is not None
            r["half"], r["stage"] = seen["src"] >> 20, (seen["src"] & 0xFFFFF) // 64
        # what the products multiply
        live = tmv[t.wave >= 4]
        count = {}
        for b, a, acc in t.products:
            assert a["stage"] == b["stage"]
            i, j = divmod(acc, 2)
            assert a["half"] == (0 if dbl else i >> 1) and b["half"] == 8 + (2 * (i >> 1) + j if dbl else j)
            assert a["addr"] % 128 // 16 == b["addr"] % 128 // 16  # the same 8 columns
            count.setdefault(acc, []).append((a["stage"], a["addr"] % 128 // 16))
        rows = [2 * h + i for h in (0, 1) for i in (0, 1) if ((0 if dbl else 2 * h) + i) < live]
        assert sorted(count) == sorted(2 * i + j for i in rows for j in (0, 1))
        for got in count.values():
            assert len(got) == len(set(got)) == 4 * (k1 - k0) and {s for s, _ in got} == set(range(k0, k1))
