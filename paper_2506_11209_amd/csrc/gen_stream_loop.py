"""Generate ws_stream_loop.inc: the K loop of one output tile for the
streaming consumer, as one asm block per kernel configuration.

    python paper_2506_11209_amd/csrc/gen_stream_loop.py            # rewrite the .inc
    python paper_2506_11209_amd/csrc/gen_stream_loop.py --check    # exit 1 if it is stale

The wave keeps F fragment sets (the operands of one k-step each) in fixed
registers at the top of the register file and reads k-step t + F - 1 while
k-step t multiplies.  A consumer wave is mostly alone on its SIMD with
producer waves, so nothing hides what it issues between its MFMAs: a wave
issues one instruction about every four clocks and a 32x32x16 MFMA takes 32,
so seven other instructions fit behind each MFMA, and a taken branch costs as
much as one.  Hence
  * the ring's bookkeeping (check of the next slot, its counter's peek, the
    addresses, the release) is spread over the MFMAs of the k-step instead of
    standing between two of them;
  * what the common case does not run (polling a slot that is not full yet,
    the delay test hook) is out of line, behind branches that are not taken;
  * the ring is walked by byte addresses (slot, full counter, empty counter)
    that wrap by compare and select, with no index arithmetic;
  * the A offset of every k-step of a slot is precomputed (the XOR swizzle),
    the B address moves once per slot.

Per k-step t of a tile (T = S KS k-steps, KS = TK / 16 per K-iteration):
  * wait for the reads of k-step t; when t is the last k-step of K-iteration
    u, every read of u has then completed and u's slot is released;
  * if k-step t + F - 1 exists, read it; when it starts a K-iteration, first
    check that K-iteration's slot is full (its counter was peeked when the
    read stream entered the slot before it) and peek at the next counter.
The release of u comes before the check of u + 2 in program order (F - 1 <=
KS + 1), so two ring slots are enough.

Twelve waves leave 168 registers a wave, 128 of them a 64 x 128 or 128 x 64
accumulator: those configurations keep one fragment set (F = 1).  The MFMAs
then run along the wave tile's longer side, so that each fragment's last use
in k-step t and its first use in k-step t + 1 are four MFMAs apart, and each
fragment is read again right behind its last use.

At KS = 4, F = 4 the check of K-iteration u + 1 stands in u's second k-step,
two before u's slot is released.  Where the slot is not full (after a second
look) and the ring has two or three slots, the block drains instead of waiting
there: it releases u's slot, whose reads have all completed, multiplies the rest
of u and then waits, so that a ring of three slots is not one of two while the
consumers wait.  It then reads u + 1 with nothing to multiply, which deeper
rings do not win back.  Waiting -> draining, 64x64x64: two slots
1024x1024x8192 75 -> 51 us, three slots 4096^3 261 -> 252 us (LDS-DMA 269 ->
241), 64x4096x4096 23.3 -> 21.3 us; 128x128x64 2048x2048x32768 three slots
286 -> 279 us, four slots 264 -> 265 us and the general kernel 277 -> 302 us.

At KS = 2 four sets read more than a slot ahead: the check of K-iteration u + 2
stands right behind the release of u, whose slot it needs in a ring of two, with
all of u + 1 still to multiply.  There a second block with two sets (tile_short)
checks u + 1 at the end of u.

The loop body is U = lcm(KS, F) k-steps, m = U / KS K-iterations.  A tile
whose S is not a multiple of m enters its first body at the k-step that makes
the rest whole (one prologue per remainder).  Tiles with S < m take the
compiler-scheduled consumer.

Every LDS wait is "at most n younger LDS operations outstanding" (a wave's
LDS operations complete in order); the generator derives each n by replaying
the emitted operations along every path through the block and keeping the
tightest, capped at 15, the counter's range.
"""
from __future__ import annotations

import math
import os
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
if HERE not in sys.path:
    sys.path.insert(0, HERE)
from gen_deep_loop import Emitter, HEADER_BYTES, LGKM_MAX  # noqa: E402

OUT = os.path.join(HERE, "ws_stream_loop.inc")

# (TM, TN, TK, NC, NP): (fragment sets F, registers a wave).  Four consumer
# waves in a 2 x 2 grid, or one.  The smallest tiles have the fewest registers:
# what hides their latency is the number of workgroups that share a CU (168 and
# 128 -> 80 registers: 32x32x32 2:1 at 1344x864x2944, two slots, 112.5 -> 41.2 us;
# 64x64x32 2:1 by four waves at 2944x960x2784 83.3 -> 50.3 us).
CONFIGS = {
    (256, 128, 64, 4, 4): (4, 256), (128, 256, 64, 4, 4): (4, 256), (128, 128, 64, 4, 4): (4, 256),
    (64, 128, 64, 4, 4): (4, 256), (128, 64, 64, 4, 4): (4, 256), (64, 64, 64, 4, 4): (4, 128),
    (128, 256, 32, 4, 4): (4, 256), (256, 128, 32, 4, 4): (4, 256), (128, 128, 32, 4, 4): (2, 128),
    (128, 128, 64, 4, 8): (4, 168), (128, 64, 64, 4, 8): (4, 168), (64, 128, 64, 4, 8): (4, 168),
    (64, 64, 64, 4, 8): (4, 168),
    (128, 128, 32, 4, 8): (4, 168), (128, 64, 32, 4, 8): (4, 168), (64, 128, 32, 4, 8): (4, 168),
    (64, 64, 32, 4, 8): (4, 168),
    (64, 128, 32, 4, 4): (4, 128), (128, 64, 32, 4, 4): (4, 128), (64, 64, 32, 4, 4): (4, 80),
    (32, 32, 32, 1, 1): (4, 128), (32, 32, 64, 1, 1): (4, 168), (64, 64, 32, 1, 1): (4, 256),
    (64, 64, 64, 1, 1): (4, 256),
    (32, 32, 32, 1, 2): (4, 80), (32, 32, 64, 1, 2): (4, 128), (64, 64, 32, 1, 2): (4, 256),
    (64, 64, 64, 1, 2): (4, 256),
    (128, 256, 32, 4, 8): (1, 168), (256, 128, 32, 4, 8): (1, 168),
    (128, 256, 64, 4, 8): (1, 168), (256, 128, 64, 4, 8): (1, 168),
}


class Cfg:
    """A configuration's block; short: the one for rings of two slots."""

    def __init__(self, tm, tn, tk, nc, np, short=False):
        assert nc in (1, 4) and tk in (32, 64)
        self.tm, self.tn, self.tk, self.nc, self.np = tm, tn, tk, nc, np
        self.f, self.vgprs = CONFIGS[(tm, tn, tk, nc, np)]
        self.ks = tk // 16
        self.has_short = self.f - 1 > self.ks
        if short:
            assert self.has_short
            self.f = 2
        self.wm, self.wn = (tm // 2, tn // 2) if nc == 4 else (tm, tn)
        self.bm, self.bn = self.wm // 32, self.wn // 32
        self.nd = tn // 32                            # B blocks (256 bytes) per block row
        self.a_bytes = tm * tk * 2
        self.stage = self.a_bytes + tk * tn * 2
        self.reads = self.bm + 2 * self.bn            # LDS instructions per fragment set
        self.set_regs = 4 * (self.bm + self.bn)
        self.frag_base = self.vgprs - self.f * self.set_regs
        self.ahead = max(1, self.f - 1)               # k-steps read ahead
        self.body = self.ks * self.f // math.gcd(self.ks, self.f)
        self.m = self.body // self.ks                 # K-iterations per loop body
        self.drain = self.f == 4 and self.ks == 4     # see the module's text
        assert self.ahead <= self.ks + 1 and self.ahead < self.body
        assert self.bm * self.bn * 16 + self.f * self.set_regs <= self.vgprs - 16
        assert self.f > 1 or sorted((self.bm, self.bn)) == [2, 4]
        assert self.stage % 128 == 0 and HEADER_BYTES % 128 == 0


def spread(mfmas, filler):
    """The MFMAs in order with the filler units evenly behind them."""
    out, done = [], 0
    for i, m in enumerate(mfmas):
        out.append(m)
        upto = (len(filler) * (i + 1) + len(mfmas) - 1) // len(mfmas)
        out += filler[done:upto]
        done = upto
    return out


def program(E: Emitter, c: Cfg, bf16: bool, S: int | None, drains=()):
    """Emit the block.  With S given (a dry run) only the path of a tile of S
    K-iterations is emitted, with absolute k-step numbers in the tags, draining
    in the loop bodies listed in `drains`; with S None every segment is emitted
    once."""
    mfma = "v_mfma_f32_32x32x16_bf16" if bf16 else "v_mfma_f32_32x32x16_f16"
    KS, F, U, m, D = c.ks, c.f, c.body, c.m, c.ahead
    emit = E.emit
    stubs = []                     # (label, kind) of out-of-line code
    drained = []                   # (k-step, MFMAs left of it) where a drain leaves the body
    dry = S is not None
    label = [20]

    def new_label():
        label[0] += 2
        return label[0]

    def a_reg(s, mb):
        b = c.frag_base + s * c.set_regs + 4 * mb
        return "v[%d:%d]" % (b, b + 3)

    def b_regs(s, nb):
        b = c.frag_base + s * c.set_regs + 4 * c.bm + 4 * nb
        return "v[%d:%d]" % (b, b + 3), "v[%d:%d]" % (b, b + 1), "v[%d:%d]" % (b + 2, b + 3)

    # Filler units: each is a list of (kind, line, tag) kept together.
    def ins(*lines):
        return [("i", l, None) for l in lines]

    def a_addr(t):
        k = t % KS
        if F == 1 and k:  # in place (registers are tight): the k-step's bits of the swizzled chunk flip
            return ins("v_xor_b32 %%[va], %d, %%[va]" % (32 * (k ^ (k - 1))))
        return ins("v_add_u32 %%[va], %%[rb], %%[ao%d]" % k)

    def read_a(t, mb):
        off = mb * 32 * c.tk * 2
        assert off < 65536
        return [[("op", "ds_read_b128 %s, %%[va] offset:%d" % (a_reg(t % F, mb), off), ("A", t, mb))]]

    def read_b(t, nb):
        _, lo, hi = b_regs(t % F, nb)
        off = ((4 * (t % KS)) * c.nd + nb) * 256
        assert off + c.nd * 256 < 65536
        return [[("op", "ds_read_b64_tr_b16 %s, %%[vb] offset:%d" % (lo, off), ("B", t, nb))],
                [("op", "ds_read_b64_tr_b16 %s, %%[vb] offset:%d" % (hi, off + c.nd * 256), ("B", t, nb))]]

    def reads(t):
        units = [a_addr(t)]
        for mb in range(c.bm):
            units += read_a(t, mb)
        for nb in range(c.bn):
            units += read_b(t, nb)
        return units

    def mf(t, mb, nb):
        s = t % F
        return ins("%s %%[c%d_%d], %s, %s, %%[c%d_%d]" % (mfma, mb, nb, a_reg(s, mb), b_regs(s, nb)[0], mb, nb))

    def mfmas(t):
        return [mf(t, mb, nb) for mb in range(c.bm) for nb in range(c.bn)]

    def of_kstep(t):
        return lambda tag: tag[0] in ("A", "B") and tag[1] == t

    def peek(u):
        # (fa, rt) <- counter address and target of K-iteration u, and read it
        return [ins("s_add_u32 %[fa], %[fa], 4", "s_cmp_eq_u32 %[fa], %[fend]",
                    "s_cselect_b32 %%[t0], %d, 0" % c.np, "s_cselect_b32 %[fa], %[fullb], %[fa]"),
                ins("s_add_u32 %[rt], %[rt], %[t0]", "v_mov_b32 %[vx], %[fa]"),
                [("op", "ds_read_b32 %[vp], %[vx]", ("peek", u))]]

    def next_slot():
        return ins("s_add_u32 %%[rb], %%[rb], %d" % c.stage, "s_cmp_eq_u32 %[rb], %[rend]",
                   "s_cselect_b32 %[rb], %[ring], %[rb]")

    def enter(site, u):
        # the read stream moves on to K-iteration u > 0
        k = new_label()
        stubs.append((k, "drain" if c.drain and site[0] == "body" else "poll"))
        stubs.append((k + 1000, "delay"))
        return [[("wait", site, ("peek", u))] + ins("v_readfirstlane_b32 %[t0], %[vp]"),
                ins("s_sub_u32 %[t0], %[t0], %[rt]", "s_cmp_lt_i32 %[t0], 0", "s_cbranch_scc1 %df" % k,
                    "%d:" % (k + 1)),
                ins("s_cmp_lg_u32 %[dly], 0", "s_cbranch_scc1 %df" % (k + 1000), "%d:" % (k + 1001)),
                next_slot(), ins("v_add_u32 %[vb], %[rb], %[boff]")] + peek(u + 1)

    def release(u):
        # K-iteration u's slot back to the producers: its reads have completed
        return [ins("v_mov_b32 %[vx], %[ea]"),
                ins("s_mov_b64 exec, 1") + [("op", "ds_add_u32 %[vx], %[one]", ("rel", u))] +
                ins("s_mov_b64 exec, -1"),
                ins("s_add_u32 %[ea], %[ea], 4", "s_cmp_eq_u32 %[ea], %[eend]",
                    "s_cselect_b32 %[ea], %[emptyb], %[ea]")]

    def put(unit):
        for kind, a, tag in unit:
            if kind == "i":
                emit(a)
            elif kind == "op":
                E.op(a, tag)
            else:
                E.wait_for(a, lambda x, tag=tag: x == tag)

    def kstep_single(seg, j, t, read_ahead):
        # F = 1: k-step t, its fragments read again for t + 1 behind their last use
        last = t % KS == KS - 1
        long_m = c.bm > c.bn        # along the longer side of the wave tile
        n_out, n_in = (c.bn, c.bm) if long_m else (c.bm, c.bn)
        if read_ahead and last:
            head = enter((seg, j, "enter"), (t + 1) // KS)
        else:
            head = []
        if read_ahead:
            head = head + [a_addr(t + 1)]
        first = n_in  # MFMAs of the first run, which the head is spread behind
        i = 0
        for o in range(n_out):
            for x in range(n_in):
                mb, nb = (x, o) if long_m else (o, x)
                E.wait_for((seg, j, "use", i), lambda tag, mb=mb, nb=nb: tag in (("A", t, mb), ("B", t, nb)))
                put(mf(t, mb, nb))
                if o == 0:
                    for unit in head[len(head) * x // first:len(head) * (x + 1) // first]:
                        put(unit)
                if last and o == n_out - 1 and x == 0:
                    E.wait_for((seg, j, "rel"), of_kstep(t))
                    for unit in release(t // KS):
                        put(unit)
                units = []
                if read_ahead and x == n_in - 1:   # the fragment of this run
                    units += read_b(t + 1, o) if long_m else read_a(t + 1, o)
                if read_ahead and o == n_out - 1:  # the fragment shared by the runs
                    shared = read_a(t + 1, x) if long_m else read_b(t + 1, x)
                    units = shared + units
                for unit in units:
                    put(unit)
                i += 1

    def kstep(seg, j, t, read_ahead):
        # k-step t (position j in the body)
        if F == 1:
            kstep_single(seg, j, t, read_ahead)
            return
        E.wait_for((seg, j, "R"), of_kstep(t))
        filler = []
        if t % KS == KS - 1:
            filler += release(t // KS)
        if read_ahead:
            if (t + D) % KS == 0:
                filler += enter((seg, j, "enter"), (t + D) // KS)
            filler += reads(t + D)
        units = spread(mfmas(t), filler)
        if c.drain and seg == "body" and (t + D) % KS == 0:
            at = next(i for i, unit in enumerate(units) if any("s_cbranch" in x[1] for x in unit))
            rest = [unit for unit in units[at + 1:] if "v_mfma" in unit[0][1]]
            if dry and t // U in drains:
                for unit in units[:at + 1]:
                    put(unit)
                drain(t, rest)
                return True
            drained.append((t, rest))
        for unit in units:
            put(unit)
        return False

    def drain(t, rest):
        # The slot of the K-iteration to enter, u, is not full.  Every read so
        # far has completed: release the slot of u - 1, multiply its k-steps
        # t (what is left of it) .. t + D - 1, and only then wait for u and
        # read its first D k-steps, which is the state at the body's start.
        u = (t + D) // KS
        E.ops.clear()
        emit("s_waitcnt lgkmcnt(0)")  # the second look's wait, again on the release's own straight line
        for unit in release(u - 1):
            put(unit)
        for unit in rest + [m for x in range(t + 1, t + D) for m in mfmas(x)]:
            put(unit)
        if not dry:
            poll(2900, 2901)
        put(next_slot())
        put(ins("v_add_u32 %[vb], %[rb], %[boff]"))
        for unit in peek(u + 1):
            put(unit)
        for x in range(t + D, t + 2 * D):
            for unit in reads(x):
                put(unit)

    def poll(again, full):
        # poll K-iteration u's counter (address fa, target rt) until it is full
        emit("s_mov_b32 %[spins], 0")
        emit("%d:" % again)
        emit("v_mov_b32 %[vx], %[fa]")
        emit("ds_read_b32 %[vp], %[vx]")
        emit("v_mov_b32 %[vx], %[abortb]")
        emit("ds_read_b32 %[vx], %[vx]")
        emit("s_waitcnt lgkmcnt(0)")
        emit("v_readfirstlane_b32 %[t0], %[vp]")
        emit("s_sub_u32 %[t0], %[t0], %[rt]")
        emit("s_cmp_ge_i32 %[t0], 0")
        emit("s_cbranch_scc1 %d%s" % (full, "f" if full == again + 1 else "b"))
        emit("v_readfirstlane_b32 %[t0], %[vx]")
        emit("s_mov_b32 %[st], 1")
        emit("s_cmp_lg_u32 %[t0], 0")
        emit("s_cbranch_scc1 9b")
        emit("s_add_u32 %[spins], %[spins], 1")
        emit("s_mov_b32 %[st], 2")
        emit("s_cmp_gt_i32 %[spins], %[lim]")
        emit("s_cbranch_scc1 9b")
        emit("s_mov_b32 %[st], 0")
        emit("s_sleep 1")
        emit("s_branch %db" % again)
        if full == again + 1:
            emit("%d:" % full)

    def prologue(j0):
        # reads of the tile's first D k-steps, which sit at body position j0 ..
        for t in range(j0, j0 + D):
            if t > j0 and t % KS == 0:
                for unit in enter(("pro", j0, t, "enter"), t // KS):
                    put(unit)
            for unit in reads(t):
                put(unit)

    # entry: the caller has waited for the tile's first slot (rb, fa, rt); the
    # accumulators were just written by VALU instructions.  K-iterations are
    # numbered from the first body's first, so that k-step t uses set t mod F.
    emit("s_nop 7")
    emit("s_mov_b32 %[st], 0")
    emit("v_mov_b32 %[one], 1")
    emit("v_add_u32 %[vb], %[rb], %[boff]")
    rems = [0] if S is None else [S % m]
    j0s = {r: ((m - r) % m) * KS for r in range(m)}

    def kk(extra):
        # loop bodies before the last one: (S + extra) / m - 1
        emit("s_add_u32 %%[kk], %%[S], %d" % extra)
        assert m & (m - 1) == 0, "loop bodies are counted by a shift"
        emit("s_lshr_b32 %%[kk], %%[kk], %d" % (m.bit_length() - 1))
        emit("s_sub_u32 %[kk], %[kk], 1")

    def start(r):
        j0 = j0s[r]
        for unit in peek(j0 // KS + 1):
            put(unit)
        prologue(j0)
        kk(j0 // KS)

    if not dry:
        if m == 2:
            emit("s_bitcmp1_b32 %[S], 0")
            emit("s_cbranch_scc1 12f")
        start(0)
        emit("s_cmp_eq_u32 %[kk], 0")
        emit("s_cbranch_scc1 8f")
        emit("1:")
        for j in range(U):
            if m == 2 and j == KS:
                emit("11:")
            kstep("body", j, j, True)
        emit("13:")
        emit("s_sub_u32 %[kk], %[kk], 1")
        emit("s_cmp_lg_u32 %[kk], 0")
        emit("s_cbranch_scc1 1b")
        emit("8:")
        for j in range(U):
            kstep("tail", j, j, j + D < U)
    else:
        r = rems[0]
        j0 = j0s[r]
        start(r)
        n = (S * KS + j0) // U
        for b in range(n):
            for j in range(U):
                t = b * U + j
                if t >= j0 and kstep("tail" if b == n - 1 else "body", j, t, b < n - 1 or j + D < U):
                    break
    # the next tile's first slot; its counter and target are in fa and rt
    for l in next_slot():
        emit(l[1])
    emit("9:")
    # the peek of the next tile's counter (or reads left by an abort) may
    # still be in flight, and the caller reads the accumulators with VALU
    # instructions
    emit("s_waitcnt lgkmcnt(0)")
    for _ in range(3):
        emit("s_nop 15")
    if dry:
        return
    emit("s_branch 19f")
    if m == 2:
        emit("12:")
        start(1)
        emit("s_branch 11b")
    i = 0
    while i < len(stubs):
        k, kind = stubs[i]
        i += 1
        emit("%d:" % k)
        if kind == "delay":
            emit("s_mov_b32 %[t0], %[dly]")
            emit("%d:" % (k + 2000))
            emit("s_sleep 127")
            emit("s_sub_u32 %[t0], %[t0], 1")
            emit("s_cmp_lg_u32 %[t0], 0")
            emit("s_cbranch_scc1 %db" % (k + 2000))
            emit("s_branch %db" % (k + 1))
            continue
        if kind == "drain":
            # one more look, then drain if the ring has at most three slots
            emit("v_mov_b32 %[vx], %[fa]")
            emit("ds_read_b32 %[vp], %[vx]")
            emit("s_waitcnt lgkmcnt(0)")
            emit("v_readfirstlane_b32 %[t0], %[vp]")
            emit("s_sub_u32 %[t0], %[t0], %[rt]")
            emit("s_cmp_ge_i32 %[t0], 0")
            emit("s_cbranch_scc1 %db" % (k + 1))
            emit("s_sub_u32 %[t0], %[rend], %[ring]")
            emit("s_cmp_gt_u32 %%[t0], %d" % (3 * c.stage))
            emit("s_cbranch_scc1 2990f")
            (t, rest), = drained  # one such site per block
            drain(t, rest)
            emit("s_branch 13b")
            emit("2990:")
            poll(2950, k + 1)
            continue
        poll(k + 2000, k + 1)
    emit("19:")


def tile_iters(c: Cfg):
    """K-iterations per tile replayed by the dry runs: every remainder with no
    loop body up to three."""
    return list(range(c.m, 5 * c.m))


def gen_block(c: Cfg, bf16: bool) -> list[str]:
    waits = {}
    for S in tile_iters(c):
        for drains in ((), range(0, 9, 2), range(1, 9, 2), range(9)) if c.drain else ((),):
            E = Emitter()
            program(E, c, bf16, S, drains)
            for site, n in E.need.items():
                waits[site] = min(waits.get(site, LGKM_MAX), n)
    E = Emitter(waits)
    program(E, c, bf16, None)
    return E.lines


def gen_tile(c: Cfg, bf16: bool, name: str) -> str:
    # Every in/out operand is early-clobber: the block writes it long before it
    # last reads its inputs, and the cursor starts out equal to some of them
    # (slot and ring, full and full0, empty and empty0), which would else let
    # the compiler give both one register.
    lines = gen_block(c, bf16)
    acc_ops = ", ".join('[c%d_%d] "+&v"(c[%d][%d])' % (mb, nb, mb, nb) for mb in range(c.bm) for nb in range(c.bn))
    ao = ", ".join('[ao%d] "v"(a_off[%d])' % (k, k) for k in range(c.ks if c.f > 1 else 1))
    clobbers = ", ".join('"v%d"' % r for r in range(c.frag_base, c.vgprs))
    body = "\n".join('        "%s\\n\\t"' % l for l in lines)
    return """  static __device__ __forceinline__ uint32_t %(name)s(f32x16_t (&c)[%(bm)d][%(bn)d], const uint32_t (&a_off)[%(ks)d],
                                                  uint32_t boff, RingCursor& r, uint32_t S, int32_t lim,
                                                  int32_t dly) {
#if defined(__HIP_DEVICE_COMPILE__)
    uint32_t st, kk, t0, spins, va, vb, vp, vx, one;
    asm volatile(
%(body)s
        : %(acc)s, [rb] "+&s"(r.slot), [fa] "+&s"(r.full), [rt] "+&s"(r.target), [ea] "+&s"(r.empty),
          [st] "=&s"(st), [kk] "=&s"(kk), [t0] "=&s"(t0), [spins] "=&s"(spins), [va] "=&v"(va),
          [vb] "=&v"(vb), [vp] "=&v"(vp), [vx] "=&v"(vx), [one] "=&v"(one)
        : %(ao)s, [boff] "v"(boff), [S] "s"(S), [ring] "s"(r.ring), [rend] "s"(r.ring_end),
          [fullb] "s"(r.full0), [fend] "s"(r.full_end), [emptyb] "s"(r.empty0), [eend] "s"(r.empty_end),
          [abortb] "s"(r.abort_flag), [lim] "s"(lim), [dly] "s"(dly)
        : "memory", "scc", %(clobbers)s);
    return st;
#else
    (void)c; (void)a_off; (void)boff; (void)r; (void)S; (void)lim; (void)dly;
    return 0;
#endif
  }
""" % dict(name=name, bm=c.bm, bn=c.bn, ks=c.ks, body=body, acc=acc_ops, ao=ao, clobbers=clobbers)


def gen_struct(t, bf16: bool) -> str:
    c = Cfg(*t)
    blocks = [gen_tile(c, bf16, "tile")]
    if c.has_short:
        blocks.append(gen_tile(Cfg(*t, short=True), bf16, "tile_short"))
    return """template <>
struct StreamLoop<%d, %d, %d, %d, %d, %s> {
  static constexpr bool kAvailable = true;
  static constexpr int kMinIters = %d;  // fewest K-iterations of a tile
  static constexpr int kVgprs = %d;
  static constexpr bool kShort = %s;  // tile_short is the block for two slots
%s};
""" % (*t, "true" if bf16 else "false", c.m, c.vgprs, "true" if c.has_short else "false", "\n".join(blocks))


def generate() -> str:
    parts = ["// generated by paper_2506_11209_amd/csrc/gen_stream_loop.py -- do not edit",
             "// The K loop of one output tile for the streaming consumer (consumer_stream",
             "// in ws_gemm_kernel.hpp), one asm block per kernel configuration.",
             "",
             "template <int TM, int TN, int TK, int NC, int NP, bool BF16>",
             "struct StreamLoop {",
             "  static constexpr bool kAvailable = false;",
             "  static constexpr int kMinIters = 1;",
             "  static constexpr int kVgprs = 0;",
             "  static constexpr bool kShort = false;",
             "};",
             ""]
    for t in CONFIGS:
        for bf16 in (True, False):
            parts.append(gen_struct(t, bf16))
    return "\n".join(parts)


def main(argv=None):
    argv = sys.argv[1:] if argv is None else argv
    text = generate()
    if "--check" in argv:
        with open(OUT) as f:
            same = f.read() == text
        print("ws_stream_loop.inc is %s" % ("up to date" if same else "STALE"))
        return 0 if same else 1
    with open(OUT, "w") as f:
        f.write(text)
    print("wrote", OUT)
    return 0


if __name__ == "__main__":
    sys.exit(main())
