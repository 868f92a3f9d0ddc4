"""Host-side model of the LDS ring protocols of the matrix-product kernels (no GPU, no library).

The kernels track their global -> LDS copies with a counter of copies in flight (a wait for "all but the
last n" completes the older ones, in issue order) and one workgroup barrier per K tile.  This test replays
the order of issues, waits, barriers and fragment reads that the kernel sources spell out, those of the default calls and those
of the fixed configurations, and checks the
two properties the protocol exists for, for every number of K tiles from 1 to 40:

  * every copy of a stage has been waited for, by the wave that issued it, before the barrier that
    precedes the first read of that stage (all waves run the same sequence, so one wave stands for all);
  * a ring slot is overwritten only by a copy issued after the barrier that follows the last read of the
    stage it held.

The literal wait expressions the model assumes are also looked up in the sources, so that a change of the
kernel without a change of the model fails here.
"""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_14719_amd", "csrc")


class Wave:
    """The copy bookkeeping of one wave: issue order, what has been waited for, what each slot holds."""

    def __init__(self, stages):
        self.stages = stages
        self.issued = []            # (stage, piece, tile during which it was issued; -1 = prologue)
        self.complete = 0           # the first `complete` issued copies are known to have landed
        self.slot_stage = {}        # slot -> stage of the copy most recently issued into it

    def issue(self, stage, piece, tile, last_read_tile_of):
        slot = stage % self.stages
        prev = self.slot_stage.get(slot)
        if prev is not None and prev != stage:
            # the stage that sat in this slot must not be read any more: its reads end with tile
            # last_read_tile_of(prev), and this copy is issued during `tile`, after that tile's successor's barrier
            assert last_read_tile_of(prev) < tile, "slot %d: stage %d overwritten during tile %d while stage %d is still read" % (slot, stage, tile, prev)
        self.slot_stage[slot] = stage
        self.issued.append((stage, piece, tile))

    def wait(self, n):
        self.complete = max(self.complete, len(self.issued) - n)

    def stage_complete(self, stage):
        idx = [i for i, c in enumerate(self.issued) if c[0] == stage]
        return bool(idx) and max(idx) < self.complete


def run_paired(nk, lpg):
    """Five stages; even tiles issue stages j+4 and j+5 alternately, one copy per slot; the fragments of tile
    j+1 are read during tile j; waits: all but 2*lpg (even j) or all but 2*lpg+1 (odd j)."""
    w = Wave(5)
    clamp = lambda s: min(s, nk - 1)
    # a stage s is read as "fragments of tile s": during tile s-1 (stage 0: in the prologue); the last tile re-reads itself
    last_read = lambda s: s - 1 if s < nk else -1          # stages past the end are never read
    for s in range(4):
        for i in range(lpg):
            w.issue(s, i, -1, last_read)
    w.wait(3 * lpg)
    assert w.stage_complete(0)
    for j in range(nk):
        w.wait(2 * lpg if j % 2 == 0 else 2 * lpg + 1)
        # barrier j: every wave has waited as above, so stage min(j+1, nk-1) must be complete
        assert w.stage_complete(clamp(j + 1)), "tile %d of %d: stage %d read before its copies were waited for" % (j, nk, clamp(j + 1))
        if j % 2 == 0:
            for q in range(2 * lpg):
                w.issue(j + 4 + (q & 1), q >> 1, j, last_read)
    w.wait(0)
    return len(w.issued)


def run_unpaired(nk, lpg, stages):
    """`stages` stages, copies stages-1 tiles ahead, one stage per tile; steady-state wait: all but
    (ahead-2)*lpg; draining tiles wait for what is left."""
    ahead = stages - 1
    w = Wave(stages)
    last_read = lambda s: s - 1
    for s in range(min(ahead, nk)):
        for i in range(lpg):
            w.issue(s, i, -1, last_read)
    w.wait((min(ahead, nk) - 1) * lpg)
    assert w.stage_complete(0)
    for j in range(nk):
        steady = j + ahead < nk
        if steady:
            w.wait((ahead - 2) * lpg)
        elif ahead > 3 and j + 3 < nk:
            w.wait(2 * lpg)
        elif j + 2 < nk:
            w.wait(lpg)
        else:
            w.wait(0)
        if j + 1 < nk:
            assert w.stage_complete(j + 1), "tile %d of %d: stage %d not complete" % (j, nk, j + 1)
        if j + ahead < nk:
            for i in range(lpg):
                w.issue(j + ahead, i, j, last_read)
    assert w.complete == len(w.issued)
    return len(w.issued)


@pytest.mark.parametrize("lpg", [4, 8])              # 8 waves: 4 copies per wave and stage; 4 waves: 8
def test_paired_ring(lpg):
    for nk in range(1, 41):
        n = run_paired(nk, lpg)
        assert n == 4 * lpg + ((nk + 1) // 2) * 2 * lpg


@pytest.mark.parametrize("stages", [4, 5])
@pytest.mark.parametrize("lpg", [4, 8])
def test_unpaired_ring(lpg, stages):
    for nk in range(1, 41):
        assert run_unpaired(nk, lpg, stages) == nk * lpg


# ------------------------------------------------------------ the kernels behind the default calls (gemm_nt_tile_kernel.hip)
def run_tile_kernel(nk, nfull, S, ppw, short_wait=0):
    """S stages; the fragments of stage j are read during tile j - 1 (stage 0: in the prologue) and have arrived before
    barrier j; the copies of stage j + S go out behind barrier j."""
    w = Wave(S)
    last_read = lambda s: s - 1
    wait_out = lambda out: w.wait({2: 2 if S > 3 else 0, 1: 1 if S > 2 else 0}.get(out, 0) * ppw)
    for s in range(min(S, nk)):
        for i in range(ppw):
            w.issue(s, i, -1, last_read)
    if nk >= S:
        w.wait((S - 1) * ppw)
    else:
        wait_out(nk - 1)
    assert w.stage_complete(0)

    def tile(j, steady):
        assert not steady or j + S < nfull                 # its copies are of a whole stage
        if steady:
            w.wait((S - 2) * ppw + short_wait)
        else:
            wait_out(min(S - 2, nk - 2 - j))
        if j + 1 < nk:
            assert w.stage_complete(j + 1), "tile %d of %d: stage %d read before its copies were waited for" % (j, nk, j + 1)
        if steady or j + S < nk:
            for i in range(ppw):
                w.issue(j + S, i, j, last_read)

    j = 0
    while j + 1 + S < nfull:
        tile(j, True)
        tile(j + 1, True)
        j += 2
    while j < nk:
        tile(j, False)
        j += 1
    assert w.complete == len(w.issued) == nk * ppw         # the epilogue reuses the ring


@pytest.mark.parametrize("S,ppw", [(4, 2), (4, 4), (2, 8)])   # 64 x 64 (16-bit, E4M3), 128 x 128 in pairs, 128 x 128 as the second
def test_tile_kernel_ring(S, ppw):
    for nk in range(1, 41):
        for nfull in (nk, nk - 1):                         # a whole last stage, and one that is half filled
            run_tile_kernel(nk, nfull, S, ppw)
    with pytest.raises(AssertionError):
        run_tile_kernel(40, 40, S, ppw, short_wait=1)


def run_wide_kernel(nk, nfull, ppw=8, slots=5, short_wait=0, swap_free=False):
    """Five slots for the operand tiles A_0 B_0 A_1 B_1 A_2 ...; behind the barrier of step p (all of step p has been read)
    B_{p+2} and then A_{p+3} go into the slots of A_p and B_p while step p + 1 is read."""
    content, issued, complete = {}, [], 0                  # slot -> operand tile; copies in issue order; how many are known to have landed
    reading = set()                                        # what may be read until the next barrier

    def issue(tile, slot):
        assert content.get(slot) not in reading, "%s overwritten by %s while it is read" % (content.get(slot), tile)
        content[slot] = tile
        issued.extend([tile] * ppw)

    def landed(tile):
        return tile in issued and max(i for i, t in enumerate(issued) if t == tile) < complete

    for s in range(3):
        if s < nk:
            issue(("A", s), 2 * s)
            if s < 2:
                issue(("B", s), 2 * s + 1)
    complete = max(complete, len(issued) - (3 * ppw if nk > 2 else 2 * ppw if nk > 1 else 0))
    assert landed(("A", 0)) and landed(("B", 0))
    reading = {("A", 0), ("B", 0)}
    sa = 0
    nxt = lambda s, by: (s + by) % slots

    def span(p, steady):
        nonlocal complete, sa, reading
        assert not steady or p + 3 < nfull                 # its copies are of whole steps
        complete = max(complete, len(issued) - (ppw + short_wait if steady or p + 2 < nk else 0))
        for m in "AB":
            assert landed((m, p + 1)), "step %d of %d: %s_%d read before its copies were waited for" % (p, nk, m, p + 1)
        free_a, free_b = sa, nxt(sa, 1)
        if swap_free:
            free_b = nxt(sa, 2)
        sa = nxt(sa, 2)
        assert content[sa] == ("A", p + 1) and content[nxt(sa, 1)] == ("B", p + 1)
        reading = {("A", p + 1), ("B", p + 1)}
        if steady or p + 2 < nk:
            issue(("B", p + 2), free_a)
        if steady or p + 3 < nk:
            issue(("A", p + 3), free_b)

    p = 0
    while p + 3 < nfull:
        span(p, True)
        p += 1
    while p + 1 < nk:
        span(p, False)
        p += 1
    assert len(issued) == 2 * nk * ppw                     # everything was copied; the last wait is for all of it


def test_wide_kernel_ring():
    for nk in range(1, 41):
        for nfull in (nk, nk - 1):
            if nfull >= 1:                                 # (the launcher takes no other)
                run_wide_kernel(nk, nfull)
    for broken in ({"short_wait": 1}, {"swap_free": True}):
        with pytest.raises(AssertionError):
            run_wide_kernel(40, 40, **broken)


def test_narrow_kernel_ring():
    for nk in range(1, 41):
        run_tile_kernel(nk, nk, 4, 2)
    src = open(os.path.join(CSRC, "gemm_nt_narrow_kernel.hip")).read()
    for needle in [
            "constexpr int NARROW_STAGES = 4;", "NW = 8, PPW = 2, S = NARROW_STAGES;",
            "for (int s = 0; s < S; ++s)\n        if (s < nk) issue(s);\n    wait_out(min(S - 1, nk - 1));",
            "if (out == 3) wait_vmcnt<3 * PPW>();\n        else if (out == 2) wait_vmcnt<2 * PPW>();\n        else if (out == 1) wait_vmcnt<1 * PPW>();\n        else wait_vmcnt<0>();",
            "if (STEADY) wait_vmcnt<(S - 2) * PPW>(); else wait_out(min(S - 2, nk - 2 - j));\n        __builtin_amdgcn_s_waitcnt(0xC07F);     // lgkmcnt(0)\n        ring_barrier();",
            "if (STEADY || j + S < nk) issue(j + S);", "for (; j + 1 + S < nk; j += 2) {"]:
        assert needle in src, "gemm_nt_narrow_kernel.hip no longer contains `%s`" % needle


def test_default_kernels_spell_out_the_waits_the_model_assumes():
    src = open(os.path.join(CSRC, "gemm_nt_tile_kernel.hip")).read()
    for needle in [
            # the kernel with S stages
            "if (nk >= S) wait_vmcnt<(S - 1) * PPW>(); else wait_out(nk - 1);",
            "if (STEADY) wait_vmcnt<(S - 2) * PPW>(); else wait_out(min(S - 2, nk - 2 - j));",
            "if (S > 3 && out == 2) wait_vmcnt<(S > 3 ? 2 : 0) * PPW>();",
            "else if (S > 2 && out == 1) wait_vmcnt<(S > 2 ? 1 : 0) * PPW>();",
            "const bool copy = STEADY || j + S < nk, next = STEADY || j + 1 < nk;",
            "if (STEADY) issue_piece(j + S, i); else issue_piece_any(j + S, i);",
            "lds_base + (s % S) * STAGE_BYTES + (wave * PPW + i) * 1024",
            "} while (j + 1 + S < nfull);",
            # the kernel with five slots
            "if (nk > 2) wait_vmcnt<3 * PPW>(); else if (nk > 1) wait_vmcnt<2 * PPW>(); else wait_vmcnt<0>();",
            "copy(A, a_off, s, i, 2 * s, no_t());",
            "copy(B, b_off, s, i, 2 * s + 1, no_t());",
            "if (STEADY || p + 2 < nk) wait_vmcnt<PPW>(); else wait_vmcnt<0>();   // own copies of step p + 1",
            "const int free_a = sa, free_b = next_slot(sa, 1);",
            "sa = next_slot(sa, 2);",
            "if (STEADY || p + 2 < nk) copy(B, b_off, p + 2, i, free_a, steady);",
            "if (STEADY || p + 3 < nk) copy(A, a_off, p + 3, i - PPW, free_b, steady);",
            "do { span(p, yes_t()); } while (++p + 3 < nfull);",
            "do { span(p, no_t()); } while (++p + 1 < nk);"]:
        assert needle in src, "gemm_nt_tile_kernel.hip no longer contains `%s`" % needle
    # the wave waits for its own reads before either barrier
    assert len(re.findall(r"__builtin_amdgcn_s_waitcnt\(0xC07F\);[^\n]*\n\s*ring_barrier\(\);", src)) == 3
    # the instances: stages 4, 2, 4 with the pieces per wave of the model
    assert "launch_tile<IN, OUT, 64, 64, 2, 2, F8 ? 1 : 2, 4, 2>" in src and "launch_tile<IN, OUT, 128, 128, 2, 2, 1, 2, 2>" in src
    assert "launch_tile<IN, OUT, 128, 128, F8 ? 4 : 2, 2, F8 ? 1 : 2, 4, 1>" in src and "constexpr int SLOT = 256 * 128, SLOTS = 5;" in src


def test_model_detects_a_short_wait_and_an_early_overwrite():
    # the same replay with one copy fewer waited for, or with the pair issued one tile early, must fail
    w = Wave(5)
    last_read = lambda s: s - 1
    for s in range(4):
        for i in range(4):
            w.issue(s, i, -1, last_read)
    w.wait(3 * 4 + 1)
    assert not w.stage_complete(0)
    with pytest.raises(AssertionError):
        w2 = Wave(5)
        for s in range(5):
            for i in range(4):
                w2.issue(s, i, -1, last_read)
        w2.issue(5, 0, 0, last_read)          # slot of stage 0 during tile 0 is fine (its fragments were read in the prologue) ...
        w2.issue(6, 0, 0, last_read)          # ... but stage 1 is read during tile 0


@pytest.mark.parametrize("fname,prefix", [("gemm_nt_kernel.hip", "G_"), ("gemm_nt_fp8_kernel.hip", "H_")])
def test_sources_spell_out_the_waits_the_model_assumes(fname, prefix):
    src = open(os.path.join(CSRC, fname)).read()
    L = prefix + "LPG"
    for needle in ["wait_vmcnt<3 * %s>();" % L,
                   "if (EVEN) wait_vmcnt<2 * %s>(); else wait_vmcnt<2 * %s + 1>();" % (L, L),
                   "if (STEADY) wait_vmcnt<(%sAHEAD - 2) * %s>(); else wait_next_stage(j);" % (prefix, L),
                   "__builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): this wave's reads of stage j are complete"]:
        assert needle in src, "%s no longer contains `%s`" % (fname, needle)
    # paired issue: stage j + 4 + parity, piece index from the slot number
    assert re.search(r"issue_piece_any\(j \+ 4 \+ \(", src)
