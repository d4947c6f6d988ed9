"""Static check of the generated K loop of the streaming consumer (StreamLoop in
paper_2506_11209_amd/csrc/ws_stream_loop.inc), CPU only.

The asm text of every configuration is executed by a small interpreter on
concrete scalar values and, for several lanes of several waves, concrete LDS
addresses.  LDS operations complete in order and only when an s_waitcnt forces
them; a slot's full counter reads short for a given number of looks.  Over two
tiles in a row, for every remainder of the loop body:

  * every read lands on the lane's own element of the operand layout (computed
    here from the layout's description, not with the kernels' functions),
    inside the slot of a K-iteration already seen full and not yet released;
  * every MFMA reads registers holding exactly its k-step's, row block's and
    column block's data, and each accumulator takes its k-steps in order;
  * a slot is released once, in order, after every read of its K-iteration
    completed, and before the block waits for the K-iteration two further on
    (so two ring slots never deadlock);
  * nothing is in flight at the end, and the cursor handed back is that of the
    next tile's first K-iteration.

A wait made one weaker, a read moved ahead of its slot's check and a swapped
fragment are caught."""
import os
import re
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2506_11209_amd", "csrc")
sys.path.insert(0, CSRC)
import gen_stream_loop as gen  # noqa: E402

RING, FULL, EMPTY, ABORT = 256, 0, 32, 64


def blocks():
    with open(gen.OUT) as f:
        text = f.read()
    out = {}
    for m in re.finditer(r"struct StreamLoop<(\d+), (\d+), (\d+), (\d+), (\d+), (true|false)> \{(.*?)\n\};", text, re.S):
        key = tuple(int(x) for x in m.groups()[:5]) + (m.group(6) == "true",)
        for fn in re.finditer(r"uint32_t (tile|tile_short)\((.*?)return st;", m.group(7), re.S):
            lines = re.findall(r'^\s*"(.*)\\n\\t"$', fn.group(2), re.M)
            out[key + (fn.group(1) == "tile_short",)] = [l.strip() for l in lines]
    return out


def cfg_of(key):
    return gen.Cfg(*key[:5], short=key[6])


BLOCKS = blocks()


def swz_a(tk, r):
    return (r ^ (r >> 2)) & 3 if tk == 32 else (r ^ ((r >> 3) & 1)) & 7


class Lane:
    """A lane's operand addresses: A rows of TK elements in 16-byte chunks,
    chunk k of row r at position k ^ swz(r); B in 4 x 32 blocks of 256 bytes,
    64 bytes a row.  Lane l of an A read takes row l % 32, chunk l / 32 of the
    k-step; 16-lane group g of a B read takes k-rows 8 (g / 2) .. + 3 (and + 4)
    and column half g % 2, four lanes to a row."""

    def __init__(self, c, cw, lane):
        self.c = c
        self.row0 = (cw // 2 if c.nc == 4 else 0) * c.wm + lane % 32
        self.chunk = lane // 32
        g, j = lane // 16, lane % 16
        self.col0 = (cw % 2 if c.nc == 4 else 0) * c.wn + 16 * (g % 2) + 4 * (j % 4)
        self.krow = 8 * (g // 2) + j // 4

    def a_byte(self, kss, mb):
        r = self.row0 + 32 * mb
        return r * self.c.tk * 2 + 16 * ((2 * kss + self.chunk) ^ swz_a(self.c.tk, r))

    def b_byte(self, kss, nb, half):
        k, col = 16 * kss + self.krow + 4 * half, self.col0 + 32 * nb
        block = (k // 4) * (self.c.tn // 32) + col // 32
        return self.c.a_bytes + 256 * block + 64 * (k % 4) + 2 * (col % 32)


def vregs(tok):
    m = re.fullmatch(r"v\[(\d+):(\d+)\]", tok)
    return list(range(int(m.group(1)), int(m.group(2)) + 1)) if m else [tok]


class Bad(Exception):
    pass


class Sim:
    """polls: looks that find a slot's counter short.  dly: the consumer delay
    hook.  lim: polls before a wait gives up.  stuck: a K-iteration whose slot never
    fills.  abort_at: the K-iteration whose wait finds the workgroup's abort flag up."""

    def __init__(self, c, S, polls, P, dly=0, lim=1000, stuck=None, abort_at=None):
        self.c, self.S, self.polls, self.P = c, S, polls, P
        self.stuck, self.abort_at = stuck, abort_at
        self.sleeps = 0
        self.ahead = 0           # most K-iterations still to multiply at the check of the next one's slot
        waves = (0, 1, 2, 3) if c.nc == 4 else (0,)
        self.lanes = [Lane(c, w, l) for w in waves for l in (0, 5, 17, 38, 63)]
        self.want = [({l.a_byte(k, m): (k, m) for k in range(c.ks) for m in range(c.bm)},
                      {l.b_byte(k, n, h): (k, n, h) for k in range(c.ks) for n in range(c.bn) for h in (0, 1)})
                     for l in self.lanes]
        self.s = dict(rb=RING, fa=FULL, rt=c.np, ea=EMPTY, ring=RING, rend=RING + P * c.stage, fullb=FULL,
                      fend=FULL + 4 * P, emptyb=EMPTY, eend=EMPTY + 4 * P, abortb=ABORT, S=S, lim=lim, dly=dly)
        self.v = {"boff": [l.b_byte(0, 0, 0) for l in self.lanes]}
        for k in range(c.ks):
            self.v["ao%d" % k] = [l.a_byte(k, 0) for l in self.lanes]
        self.full = {0}          # K-iterations seen full
        self.looks = {}
        self.released = 0
        self.pending = []        # (registers, value or data tag, K-iteration) oldest first
        self.data = {}
        self.mfmas = 0
        self.acc = {}
        self.exec = -1

    def val(self, t):
        t = t.strip()
        return self.s[t[2:-1]] if t.startswith("%[") else int(t, 0)

    def vec(self, t):
        t = t.strip()
        name = t[2:-1] if t.startswith("%[") else None
        return self.v[name] if name in self.v else [self.val(t)] * len(self.lanes)

    def iteration(self, slot):
        """The K-iteration a read of `slot` sees: the latest one seen full there."""
        its = [u for u in self.full if u % self.P == slot and u >= self.released]
        if len(its) != 1:
            raise Bad("slot %d holds no K-iteration seen full" % slot)
        return its[0]

    def read(self, op, dst, name, off):
        tags = set()
        for i in range(len(self.lanes)):
            rel = self.v[name][i] + off - RING
            slot, within = rel // self.c.stage, rel % self.c.stage
            if not 0 <= slot < self.P:
                raise Bad("read outside the ring")
            u = self.iteration(slot)
            kind = op == "ds_read_b64_tr_b16"
            if within not in self.want[i][kind]:
                raise Bad("lane %d reads byte %d" % (i, within))
            tags.add((u, "B" if kind else "A") + self.want[i][kind][within])
        if len(tags) != 1:
            raise Bad("lanes disagree: %s" % tags)
        tag = tags.pop()
        if any(r < self.c.frag_base or r >= self.c.vgprs for r in vregs(dst)):
            raise Bad("read into %s" % dst)
        self.pending.append((vregs(dst), tag, tag[0]))

    def ready(self, regs):
        for dst, _, _ in self.pending:
            if set(dst) & set(regs):
                raise Bad("%s used before its read completed" % (regs,))

    def wait(self, n):
        done = self.pending[:len(self.pending) - n] if n else self.pending
        self.pending = self.pending[len(done):]
        for dst, x, _ in done:
            for r in dst:
                self.data[r] = x

    def mfma(self, args):
        c = self.c
        mb, nb = (int(x) for x in re.fullmatch(r"%\[c(\d+)_(\d+)\]", args[0]).groups())
        t = self.mfmas // (c.bm * c.bn)
        self.mfmas += 1
        u, k = divmod(t, c.ks)
        a, b = vregs(args[1]), vregs(args[2])
        self.ready(a + b)
        if [self.data.get(r) for r in a] != [(u, "A", k, mb)] * 4:
            raise Bad("A operand of k-step %d holds %s" % (t, self.data.get(a[0])))
        if [self.data.get(r) for r in b] != [(u, "B", k, nb, h) for h in (0, 0, 1, 1)]:
            raise Bad("B operand of k-step %d holds %s" % (t, self.data.get(b[0])))
        if self.acc.get((mb, nb), -1) != t - 1 or args[3] != args[0]:
            raise Bad("accumulator order")
        self.acc[(mb, nb)] = t

    def tile(self, lines):
        labels = {}
        for i, l in enumerate(lines):
            if re.fullmatch(r"\d+:", l):
                labels.setdefault(l[:-1], []).append(i)
        i, scc, steps, c, s = 0, False, 0, self.c, self.s
        while i < len(lines):
            steps += 1
            assert steps < 200000
            l = lines[i]
            op = l.split()[0]
            args = [a.strip() for a in l[len(op):].split(",")]
            i += 1
            if re.fullmatch(r"\d+:", l) or op in ("s_nop", "s_sleep"):
                self.sleeps += l == "s_sleep 127"
                continue
            if op.startswith("s_cbranch") or op == "s_branch":
                assert op in ("s_branch", "s_cbranch_scc1")
                if op == "s_branch" or scc:
                    at = labels[args[0][:-1]]
                    i = min(j for j in at if j >= i) if args[0][-1] == "f" else max(j for j in at if j < i)
                continue
            name = args[0][2:-1]
            if op == "s_waitcnt":
                self.wait(int(re.search(r"lgkmcnt\((\d+)\)", l).group(1)))
            elif op in ("ds_read_b128", "ds_read_b64_tr_b16"):
                self.read(op, args[0], args[1].split()[0][2:-1], int(re.search(r"offset:(\d+)", l).group(1)))
            elif op == "ds_read_b32":
                at = self.vec(args[1])[0]
                if at == ABORT:
                    x = int(max(self.full) + 1 == self.abort_at)
                else:
                    u = max(self.full) + 1
                    if at != FULL + 4 * (u % self.P):
                        raise Bad("looks at counter %d for K-iteration %d" % (at, u))
                    if u - self.P >= self.released and self.looks.get(u, 0) > 0:
                        raise Bad("K-iteration %d waited for while its slot is held" % u)
                    looks = self.looks[u] = self.looks.get(u, 0) + 1
                    short = looks <= (self.polls if u != self.stuck else looks)
                    x = c.np * (u // self.P + 1) - (1 if short else 0)
                self.pending.append(([args[0]], x, None))
            elif op == "ds_add_u32":
                if self.exec != 1 or self.v["one"][0] != 1 or self.vec(args[0])[0] != EMPTY + 4 * (self.released % self.P):
                    raise Bad("release of the wrong slot")
                if any(u == self.released for _, _, u in self.pending) or self.released not in self.full:
                    raise Bad("released before its reads completed")
                self.released += 1
                self.pending.append(([], None, None))
            elif op.startswith("v_mfma"):
                self.mfma(args)
            elif op == "v_readfirstlane_b32":
                self.ready([args[1]])
                s[name] = self.data[args[1]]
                u = max(self.full) + 1
                if args[1] == "%[vp]":
                    self.ahead = max(self.ahead, u - self.mfmas / (c.ks * c.bm * c.bn))
                if args[1] == "%[vp]" and s[name] >= c.np * (u // self.P + 1) and s[name] == s["rt"]:
                    self.full.add(u)
            elif op == "v_mov_b32":
                self.ready([args[0]]) if name == "vp" else None
                self.v[name] = list(self.vec(args[1]))
            elif op == "v_add_u32":
                self.v[name] = [a + b for a, b in zip(self.vec(args[1]), self.vec(args[2]))]
            elif op == "v_xor_b32":
                self.v[name] = [a ^ b for a, b in zip(self.vec(args[1]), self.vec(args[2]))]
            elif op == "s_mov_b64":
                self.exec = int(args[1])
            elif op == "s_mov_b32":
                s[name] = self.val(args[1])
            elif op in ("s_add_u32", "s_sub_u32"):
                s[name] = self.val(args[1]) + (1 if op == "s_add_u32" else -1) * self.val(args[2])
            elif op == "s_lshr_b32":
                s[name] = self.val(args[1]) >> self.val(args[2])
            elif op == "s_cselect_b32":
                s[name] = self.val(args[1]) if scc else self.val(args[2])
            elif op == "s_bitcmp1_b32":
                scc = bool(self.val(args[0]) >> self.val(args[1]) & 1)
            elif op.startswith("s_cmp"):
                a, b = self.val(args[0]), self.val(args[1])
                scc = {"s_cmp_eq_u32": a == b, "s_cmp_lg_u32": a != b, "s_cmp_lt_i32": a < b,
                       "s_cmp_ge_i32": a >= b, "s_cmp_gt_i32": a > b, "s_cmp_gt_u32": a > b}[op]
            else:
                raise AssertionError("the checker does not know %r" % l)

    def run(self, lines, tiles=2):
        c = self.c
        for t in range(1, tiles + 1):
            self.tile(lines)
            n = t * self.S
            if self.pending or self.exec != -1 or self.s["st"] != 0:
                raise Bad("in flight at the end")
            if self.released != n or self.mfmas != n * c.ks * c.bm * c.bn:
                raise Bad("%d K-iterations released, %d MFMAs" % (self.released, self.mfmas))
            if (self.s["rb"], self.s["fa"], self.s["ea"], self.s["rt"]) != (
                    RING + n % self.P * c.stage, FULL + 4 * (n % self.P), EMPTY + 4 * (n % self.P),
                    c.np * (n // self.P + 1)):
                raise Bad("cursor handed back")
            self.full.add(n)  # the caller waits for the next tile's first K-iteration


@pytest.mark.parametrize("key", sorted(BLOCKS), ids=str)
def test_block_on_every_path(key):
    c = cfg_of(key)
    for S in range(c.m, c.m + 6):
        for polls in (0, 1, 3):
            for P in (2, 3, 5):
                Sim(c, S, polls, P).run(BLOCKS[key])


@pytest.mark.parametrize("key", sorted(k for k in BLOCKS if k[5]), ids=str)
def test_delay_hook(key):
    """Every K-iteration that the block enters without draining sleeps dly times;
    the delay changes nothing else."""
    c = cfg_of(key)
    for S in range(c.m, c.m + 4):
        for polls in (0, 1):
            sim = Sim(c, S, polls, 3, dly=3)
            sim.run(BLOCKS[key])
            assert sim.sleeps == 2 * 3 * (S - 1), (S, polls)
        drained = Sim(c, S, 3, 3, dly=3)
        drained.run(BLOCKS[key])
        assert drained.sleeps == (0 if c.drain else 2 * 3 * (S - 1))


@pytest.mark.parametrize("key", sorted(k for k in BLOCKS if k[5]), ids=str)
def test_two_slots_wait_with_less_than_a_k_iteration_in_hand(key):
    """In a ring of two slots the slot that a K-iteration waits for is filled while
    the one before it multiplies: a block that waits with a whole K-iteration read
    and none of it multiplied would load and multiply in turn."""
    c = cfg_of(key)
    sim = Sim(c, c.m + 4, 0, 2)
    sim.run(BLOCKS[key])
    two_slots = key[6] or not c.has_short
    assert (sim.ahead < 1) == two_slots, sim.ahead


@pytest.mark.parametrize("key", sorted(k for k in BLOCKS if k[5]), ids=str)
def test_every_wait_gives_up(key):
    """A slot that never fills, or an abort raised by another wave, ends the block
    at that K-iteration's wait with status 2 or 1, nothing in flight, every lane
    enabled and no slot released that is still read."""
    c = cfg_of(key)
    for S in range(c.m + 1, c.m + 4):
        for P in (2, 3, 5):
            for u in range(1, S):
                for st, kw in ((2, dict(lim=4)), (1, dict(abort_at=u))):
                    sim = Sim(c, S, 0, P, stuck=u, **kw)
                    sim.tile(BLOCKS[key])
                    assert sim.s["st"] == st and not sim.pending and sim.exec == -1
                    assert max(sim.full) == u - 1 and sim.released <= u


def test_committed_file_is_what_the_generator_writes():
    assert gen.main(["--check"]) == 0
    assert set(BLOCKS) == {k + (b, short) for k in gen.CONFIGS for b in (True, False)
                           for short in ((False, True) if gen.Cfg(*k).has_short else (False,))}


def shared_register_hazards(text):
    """In/out operands of the asm statements in `text` that are written while an
    input is still to be read, without being marked early-clobber: the compiler
    may give such an operand and an input of equal value one register."""
    out = []
    for body, outs, ins in re.findall(r'asm volatile\(\n(.*?)\n\s+: (.*?)\n\s+: (.*?)\n\s+: "memory"', text, re.S):
        lines = [l.strip() for l in re.findall(r'^\s*"(.*)\\n\\t"$', body, re.M)]
        inputs = re.findall(r'\[(\w+)\] "(?:s|v)"', ins)
        last = max(i for i, l in enumerate(lines) if any("%%[%s]" % n in l for n in inputs))
        for name, mark in re.findall(r'\[(\w+)\] "\+(&?)[sv]"', outs):
            wr = [i for i, l in enumerate(lines) if re.match(r"(?:v_|s_(?!cmp|cbranch))\S+ %%\[%s\]," % name, l)]
            assert wr, name
            if not mark and wr[0] < last:
                out.append(name)
    return out


def test_operands_written_early_share_no_register_with_an_input():
    with open(gen.OUT) as f:
        text = f.read()
    assert text.count("asm volatile(") == len(BLOCKS)
    assert not shared_register_hazards(text)
    assert set(shared_register_hazards(text.replace('"+&s"', '"+s"'))) == {"rb", "fa", "rt", "ea"}


@pytest.mark.parametrize("key", sorted(k for k in BLOCKS if k[5]), ids=str)
def test_planted_mistakes_are_caught(key):
    lines, c = BLOCKS[key], cfg_of(key)

    def caught(bad):
        for S in range(c.m, c.m + 4):
            try:
                Sim(c, S, 0, 3).run(bad)
            except Bad:
                return True
        return False

    weak = [i for i, l in enumerate(lines) if l.startswith("s_waitcnt") and "(15)" not in l and "s_nop" not in lines[i + 1]]
    n = 0
    for i in weak:
        k = int(re.search(r"\((\d+)\)", lines[i]).group(1))
        n += caught(lines[:i] + ["s_waitcnt lgkmcnt(%d)" % (k + 1)] + lines[i + 1:])
    assert n >= 2, (n, len(weak))  # most waits are at the counter's cap or covered by the one before
    add = [i for i, l in enumerate(lines) if l.startswith("ds_add")]
    for i in add[:2]:
        assert caught(lines[:i] + lines[i + 1:])                     # a slot never released
    mf = [i for i, l in enumerate(lines) if l.startswith("v_mfma")]
    a, b = (next(i for i in mf if "c0_0" in lines[i]), mf[-1])
    swapped = list(lines)
    swapped[a] = re.sub(r"(v\[\d+:\d+\]), (v\[\d+:\d+\])", r"\2, \1", lines[a])
    assert caught(swapped) and b > 0
