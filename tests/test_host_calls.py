"""What the device half of the library enqueues, without a GPU: the built library runs on top of a
stand-in for the HIP runtime (tests/native/hip_recorder.cpp) that records launches, copies and events
and knows which of them are ordered behind each other.  Device pointers are made-up numbers.  Every
scenario runs in a process of its own, so that the stand-in is the only runtime the library sees."""
import ctypes
import os
import shutil
import struct
import subprocess
import sys
import threading

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

import workloads  # noqa: E402


# ---- inside the scenario's process --------------------------------------------------------------------

class Recorder:
    def __init__(self, path):
        self.so = ctypes.CDLL(path, mode=ctypes.RTLD_GLOBAL)          # in front of the runtime the library names
        for f in ("rec_stream", "rec_arg", "rec_bytes", "rec_more", "rec_new_stream", "rec_live"):
            getattr(self.so, f).restype = ctypes.c_uint64
        self.so.rec_name.restype = ctypes.c_char_p
        for f in ("rec_finish_stream", "rec_set_limit", "rec_next_at"):
            getattr(self.so, f).argtypes = [ctypes.c_uint64]
        self.so.rec_set_capturing.argtypes = [ctypes.c_uint64, ctypes.c_int]

    def stream(self):
        return int(self.so.rec_new_stream())

    def ops(self, start=0):
        s = self.so
        return [(i, s.rec_name(i).decode(), int(s.rec_stream(i)), int(s.rec_arg(i)), int(s.rec_bytes(i)))
                for i in range(start, s.rec_count())]

    def before(self, a, b):
        return bool(self.so.rec_before(a, b))

    def launches(self, start=0):
        return [o for o in self.ops(start) if o[1] not in ("copy", "event")]

    def check_tables(self):
        """No table is overwritten under a kernel that reads it: a copy onto memory that the first
        argument of an earlier launch lies in is ordered behind that launch and behind earlier copies onto
        that memory, and a launch is ordered behind the last copy onto the memory its first argument lies in.
        (Small tables are written by a kernel on the caller's stream: a copy here.)"""
        ops = self.ops()
        for i, name, _, at, size in ops:
            if name == "copy":
                for j, other, _, arg, n in ops[:i]:
                    if other not in ("copy", "event") and at <= arg < at + size:
                        assert self.before(j, i), f"copy {i} overwrites the table of {other} {j}"
                    elif other == "copy" and at < arg + n and arg < at + size:
                        assert self.before(j, i), f"copy {i} may be overwritten by the earlier copy {j}"
            elif name != "event":
                copies = [j for j, other, _, to, n in ops[:i] if other == "copy" and to <= at < to + n]
                if copies:
                    assert self.before(copies[-1], i), f"{name} {i} does not wait for the copy of its table"




def tables(desc, base, size, ld_multiple=8, off=0):
    """Made-up device addresses and leading dimensions of a matrix' tiles."""
    ptr, ld = [], []
    for _ in range(desc["replication"]):
        for r0, r1 in zip(desc["row_cuts"], desc["row_cuts"][1:]):
            for c0, c1 in zip(desc["col_cuts"], desc["col_cuts"][1:]):
                w = max(-(-(c1 - c0) // ld_multiple) * ld_multiple, 1)
                ld.append(w)
                ptr.append(base + off if r1 > r0 and c1 > c0 else None)
                base += -(-(r1 - r0) * w * size // 512) * 512 + 512
    return ptr, ld


class Product:
    """A plan and made-up tiles: `aligned` rows at multiples of 16 bytes, or packed 2-byte aligned ones."""

    def __init__(self, descs, nranks, flags=0, dtype="bf16"):
        from paper_2510_08874_amd import binding
        self.b = binding
        self.descs, self.plan = descs, binding.Plan(*descs, nranks, flags)
        self.dtype = binding.DMM_BF16 if dtype == "bf16" else binding.DMM_F32
        self.size = 2 if dtype == "bf16" else 4

    def args(self, aligned=True, where=0):
        a, b, c = self.descs
        kw = dict(ld_multiple=8) if aligned else dict(ld_multiple=1, off=self.size)
        base = (1 << 44) + (where << 40)
        return self.plan.marshal(*tables(a, base, self.size, **kw), *tables(b, base + (1 << 38), self.size, **kw),
                                 *tables(c, base + (2 << 38), 4, ld_multiple=4))

    def run(self, args, flags=0, stream=0):
        self.plan.execute_marshalled(self.dtype, args, flags, stream)


def row_col(m, k, n, p=8):
    block = workloads.block_desc
    return block(m, k, p, 1), block(k, n, 1, p), block(m, n, 4, p // 4)


def uneven(m, k, n, seed):
    cuts, desc = workloads.jittered_cuts, workloads.desc
    return (desc(m, k, cuts(m, 3, seed), cuts(k, 5, seed + 1), 3, 5), desc(k, n, cuts(k, 7, seed + 2), [0, n], 7, 1),
            desc(m, n, cuts(m, 5, seed + 3), cuts(n, 3, seed + 4), 5, 3))


def dense_calls_and_others_on_two_streams(rec):
    """One plan, its calls alternating between operands that are copied first and operands that are not,
    on two streams: a call's copies must not be made before the product that reads the copies of an
    earlier call has finished, whatever ran in between on the other stream."""
    block = workloads.block_desc
    p = Product((block(6656, 3840, 8, 8), block(3840, 5376, 8, 8), block(6656, 5376, 8, 8)), 64)
    s1, s2 = rec.stream(), rec.stream()
    for other in ("aligned", "no merge"):
        plain, flags = (p.args(), 0) if other == "aligned" else (p.args(False, 3), p.b.DMM_NO_MERGE)
        seen = []
        for args, fl, stream in ((plain, flags, s2), (p.args(False, 1), 0, s1), (plain, flags, s2), (p.args(False, 2), 0, s2)):
            at = len(rec.ops())
            p.run(args, fl, stream)
            seen.append([(o[0], o[1]) for o in rec.launches(at)])
        copied = [any(n == "pack_kernel" for _, n in call) for call in seen]
        assert copied == [False, True, False, True], seen
        last_reader, next_copy = seen[1][-1][0], seen[3][0][0]
        assert rec.before(last_reader, next_copy), f"{other}: the copies of call 1 are overwritten under its product"
        rec.check_tables()
    p.plan.destroy()
    rec.check_tables()


def destroy_waits_for_every_stream(rec):
    """A plan used on two streams gives its buffers back only when both have finished with them."""
    p = Product(row_col(1024, 512, 1024), 8)
    s1, s2 = rec.stream(), rec.stream()
    args = p.args()
    p.run(args, 0, s1)
    p.run(args, 0, s2)                       # the same tables, not ordered behind the first call
    readers = [o[0] for o in rec.launches()]
    p.plan.destroy()
    q = Product(row_col(1024, 520, 1024), 8)
    q.run(q.args(), 0, rec.stream())         # may get the same buffer for its tables
    rec.check_tables()
    mark = rec.ops()[-1][0]
    assert all(rec.before(r, mark) for r in readers)
    q.plan.destroy()


def scratch_is_not_shared_by_calls_that_overlap(rec):
    """A replicated product cut along K on one stream, the replica sum alone on another, the product again
    there: the partial tiles of the first call lie in the scratch buffer that the last one writes."""
    block = workloads.block_desc
    d = (block(512, 65536, 1, 1, replication=2), block(65536, 512, 1, 1, replication=2), block(512, 512, 1, 1, replication=2))
    p = Product(d, 2)
    s1, s2 = rec.stream(), rec.stream()
    args = p.args()
    c_ptr, c_ld = list(args[4]), list(args[5])
    p.plan.reduce_replicas(c_ptr, c_ld, 0, s2)
    p.run(args, 0, s1)
    assert p.plan.ran_k_split()
    first = [o[0] for o in rec.launches()][-1]
    p.plan.reduce_replicas(c_ptr, c_ld, 0, s2)
    at = len(rec.ops())
    p.run(args, 0, s2)
    again = rec.launches(at)[0][0]
    assert rec.before(first, again), "the scratch buffer is overwritten under the first call"
    rec.check_tables()
    p.plan.destroy()


def more_streams_than_the_plan_remembers(rec):
    """Calls on many streams, then new operands: the new tables wait for every one of the calls."""
    p = Product(row_col(1024, 512, 1024), 8)
    args = p.args()
    for _ in range(11):
        p.run(args, 0, rec.stream())
    p.run(p.args(where=1), 0, rec.stream())
    rec.check_tables()
    p.plan.destroy()


def reports_say_what_ran(rec):
    """dmm_plan_last_execute and dmm_plan_last_kernels against the launches of every kind of call."""
    cyclic = workloads.block_cyclic_desc
    s = rec.stream()

    def check(p, args, flags, kernels, merged=False, small=None, dense=False, split=False, fused=0):
        at = len(rec.ops())
        p.run(args, flags, s)
        got = [o[1] for o in rec.launches(at)]
        assert got == kernels, got
        rep = p.plan.last_execute()
        assert (bool(rep.ran_merged), bool(rep.ran_k_split), rep.ran_fused) == (merged, split, fused), (merged, split, fused)
        assert p.plan.small_tile() == small and p.plan.ran_dense() == dense, (p.plan.small_tile(), p.plan.ran_dense())

    def fine(m, k, n, flags=0):              # tiles finer than the macro-tile: the plan has a merged list
        p = Product((cyclic(m, k, 128, 128, 2, 4, 1), cyclic(k, n, 128, 128, 2, 4, 1), cyclic(m, n, 128, 128, 2, 4, 1)), 8, flags)
        assert p.plan.num_merged_items() > 0
        return p

    p = fine(700, 333, 517)
    check(p, p.args(), 0, ["small_gemm_kernel"], small=(32, 128))
    check(p, p.args(), p.b.DMM_NO_MERGE, ["grouped_gemm_kernel"])
    check(p, p.args(), 0, ["small_gemm_kernel"], small=(32, 128))
    q = fine(700, 333, 517, p.b.DMM_MERGE_ALWAYS)
    check(q, q.args(), 0, ["grouped_gemm_comp_kernel"], merged=True)
    q = fine(700, 18000, 500, p.b.DMM_MERGE_ALWAYS)
    check(q, q.args(), 0, ["grouped_gemm_comp_kernel", "sum_parts_kernel"], merged=True, split=True)
    q = Product(row_col(8192, 8192, 8192), 8)                              # no merged list
    assert q.plan.num_merged_items() == 0
    check(q, q.args(), 0, ["grouped_gemm_kernel"])
    q = Product(row_col(256, 256, 256, 4), 4, dtype="f32")                 # four waves share a tile's K
    check(q, q.args(), 0, ["small_gemm_kernel"], small=(32, 32), split=True)
    q = Product(row_col(2048, 2048, 2048), 8)
    assert q.plan.num_merged_items() == 0
    check(q, q.args(), 0, ["small_gemm_kernel"], small=(128, 128))
    assert q.plan.last_kernels().small_runs == 1
    q = Product(row_col(1024, 16384, 1024), 8)
    check(q, q.args(), 0, ["small_gemm_kernel", "small_sum_kernel"], small=(128, 128), split=True)
    assert q.plan.last_kernels().small_runs > 1
    cfg = workloads.config("cfg4")
    q = Product((cfg["A"], cfg["B"], cfg["C"]), cfg["nranks"])
    check(q, q.args(), 0, ["grouped_gemm_kernel"], fused=1)
    check(q, q.args(), q.b.DMM_SEPARATE_REDUCE, ["grouped_gemm_kernel", "reduce_replicas_kernel"])
    q = fine(8192, 8192, 8192)
    check(q, q.args(False), 0, ["pack_kernel", "grouped_gemm_comp_kernel"], merged=True, dense=True)
    check(q, q.args(False), q.b.DMM_NO_MERGE, ["grouped_gemm_kernel"])


def _pack_tables(rec, op):
    """The tables of a launch of pack_kernel: jobs, runs and tiles as lists of tuples."""
    so, n = rec.so, int(rec.so.rec_more(op, 0))
    job, run, tile = struct.Struct("<qq10i"), struct.Struct("<4i"), struct.Struct("<qq")
    jobs = [job.unpack(ctypes.string_at(rec.so.rec_arg(op) + i * job.size, job.size)) for i in range(n)]
    n_runs = max(j[6] + j[7] for j in jobs)
    runs = [run.unpack(ctypes.string_at(so.rec_more(op, 1) + i * run.size, run.size)) for i in range(n_runs)]
    return jobs, runs, lambda i: tile.unpack(ctypes.string_at(so.rec_more(op, 2) + i * tile.size, tile.size))


def _columns_of(job, runs, at):
    """What a thread of pack_kernel puts into eight columns of a copy from column `at` on, step by step as
    the kernel does it: ([(tile, column inside it) or None] * 8, [(tile, first column read, last)])."""
    rs = runs[job[6]:job[6] + job[7]]
    x = max(i for i, r in enumerate(rs) if r[0] <= at)
    start, length, tile, col = rs[x]
    off = at - start
    n, alone = length - off, x + 1 == len(rs) or rs[x + 1][0] >= at + 8
    if n <= 0 and alone:
        return [None] * 8, []
    if n >= 8 or (n > 0 and length >= 8 and alone):
        back = 0 if n >= 8 else 8 - n
        first = col + off - back
        return [(tile, first + back + e) if e + back < 8 else None for e in range(8)], [(tile, first, first + 7)]
    got, reads = [], []
    for e in range(8):
        while x + 1 < len(rs) and rs[x + 1][0] <= at + e:
            x += 1
        start, length, tile, col = rs[x]
        o = at + e - start
        got.append((tile, col + o) if o < length else None)
        if got[-1]:
            reads.append((tile, col + o, col + o))
    return got, reads


def the_copies_hold_the_k_steps_of_the_operands(rec):
    """The tables of pack_kernel, followed as the kernel follows them: every element of the copies is written
    once, holds the element of A (B) that belongs there or a zero, no read leaves a tile, and the K-segments
    begin at multiples of the macro-tile kernels' K step (32), filled up with zeros."""
    import numpy as np
    cyclic, cuts, desc = workloads.block_cyclic_desc, workloads.jittered_cuts, workloads.desc

    def uneven(m, k, n, s):
        return (desc(m, k, cuts(m, 3, s), cuts(k, 5, s + 1), 3, 5), desc(k, n, cuts(k, 7, s + 2), cuts(n, 2, s + 5), 7, 2),
                desc(m, n, cuts(m, 5, s + 3), cuts(n, 3, s + 4), 5, 3)), 15

    def blocks(m, k, n, nb, c):
        return tuple(cyclic(r, q, nb, nb, 2, 4, c) for r, q in ((m, k), (k, n), (m, n))), 8 * c

    with_empty = (desc(4100, 1030, (0, 0, 2050, 2050, 4100), (0, 3, 3, 500, 1030), 4, 4), desc(1030, 4101, (0, 500, 500, 1027, 1030), (0, 0, 1, 4101), 4, 3),
                  desc(4100, 4101, tuple(min(i * 100, 4100) for i in range(42)), tuple(min(i * 100, 4101) for i in range(43)), 2, 2))
    for (descs, p) in (uneven(8025, 2369, 4107, 77), blocks(4101, 2051, 4099, 100, 1), blocks(3001, 4099, 4102, 99, 2),
                       blocks(4099, 3333, 4104, 100, 3), (with_empty, 16)):
        q = Product(descs, p)
        a, b, c = descs
        at = len(rec.ops())
        q.run(q.args(False), 0, rec.stream())
        assert q.plan.ran_dense() and not q.plan.ran_k_split()
        op = [o[0] for o in rec.launches(at) if o[1] == "pack_kernel"][0]
        jobs, runs, tile_at = _pack_tables(rec, op)
        M, K, N, reps = a["rows"], a["cols"], b["cols"], c["replication"]
        shares = [r * K // reps for r in range(reps + 1)]
        kc = sorted(set(a["col_cuts"]) | set(b["row_cuts"]) | set(shares))
        segs = [[(k0, k1) for k0, k1 in zip(kc, kc[1:]) if shares[r] <= k0 < shares[r + 1]] for r in range(reps)]
        length = max(sum(-(-(k1 - k0) // 32) * 32 for k0, k1 in s) for s in segs)
        k_of = np.full((reps, length), -1)                                # which k a column of A's copy (a row of B's) holds
        for r, s in enumerate(segs):
            pos = length - sum(-(-(k1 - k0) // 32) * 32 for k0, k1 in s)
            for k0, k1 in s:
                assert pos % 32 == 0
                k_of[r, pos:pos + k1 - k0] = np.arange(k0, k1)
                pos += -(-(k1 - k0) // 32) * 32
        lda, ldb = -(-length // 64) * 64, -(-N // 64) * 64
        base = min(j[0] for j in jobs)
        wrote_a, wrote_b = np.zeros((reps, M), int), np.zeros(reps * length, int)
        tiles_a = (len(a["row_cuts"]) - 1) * (len(a["col_cuts"]) - 1)
        block = 0
        for j in jobs:
            dst, pitch, rows, rows_out, row, cols_out, _, _, tile0, first_block, blocks_c, _ = j[:12]
            assert dst % 16 == 0 and pitch % 16 == 0 and first_block == block and blocks_c == -(-cols_out // 2048)
            block += blocks_c * -(-rows_out // 8)
            off = dst - base
            of_a = off < 2 * reps * M * lda
            if of_a:
                rep, first_row = divmod(off // (2 * lda), M)
                assert off % (2 * lda) == 0 and pitch == 2 * lda and cols_out == length and rows == rows_out
                wrote_a[rep, first_row:first_row + rows_out] += 1
                G, where = a, tile0
                ti, left = divmod(where, len(a["col_cuts"]) - 1)
                assert left == 0 and a["row_cuts"][ti] + row == first_row and rows <= a["row_cuts"][ti + 1] - first_row
            else:
                first_row, left = divmod(off - 2 * reps * M * lda, 2 * ldb)
                assert left == 0 and pitch == 2 * ldb and cols_out == N
                wrote_b[first_row:first_row + rows_out] += 1
                held = k_of.reshape(-1)[first_row:first_row + rows_out]
                G, where = b, tile0 - tiles_a
                ti, left = divmod(where, len(b["col_cuts"]) - 1)
                assert left == 0 and (held[rows:] == -1).all()
                if rows:
                    assert (held[:rows] == b["row_cuts"][ti] + row + np.arange(rows)).all() and held[0] + rows <= b["row_cuts"][ti + 1]
            if rows == 0:
                continue
            cc = G["col_cuts"]
            for col in range(0, cols_out, 8):
                got, reads = _columns_of(j, runs, col)
                for tile, lo, hi in reads:
                    assert 0 <= lo and hi < cc[tile + 1] - cc[tile], "a read leaves its tile"
                    ptr, src_pitch = tile_at(tile0 + tile)
                    assert ptr and src_pitch == 2 * (cc[tile + 1] - cc[tile])
                for e, g in enumerate(got):
                    want = k_of[rep, col + e] if of_a and col + e < length else col + e if not of_a and col + e < N else -1
                    assert (cc[g[0]] + g[1] if g else -1) == want
        assert block == rec.so.rec_blocks(op) and (wrote_a == 1).all() and (wrote_b == 1).all()
        q.plan.destroy()


def copies_do_not_show_in_the_bits(rec):
    """Whether a call takes the copies depends on where its operands lie and on free memory; its bits must not.
    What runs on copies is never cut along K, and then neither is what runs in their place."""
    import random
    rng, cyclic, cuts, desc = random.Random(11), workloads.block_cyclic_desc, workloads.jittered_cuts, workloads.desc
    dense = was_cut = 0
    problems = []
    for _ in range(60):
        m, k, n = rng.randrange(5000, 9000), rng.randrange(6500, 16000), rng.randrange(5000, 9000)    # copies of 130 MB and more
        if rng.random() < 0.5:
            s = rng.randrange(1000)
            descs, p = (desc(m, k, cuts(m, 3, s), cuts(k, 5, s + 1), 3, 5), desc(k, n, cuts(k, 7, s + 2), (0, n), 7, 1),
                        desc(m, n, cuts(m, 5, s + 3), cuts(n, 3, s + 4), 5, 3)), 15
        else:
            c, nb = rng.choice((1, 2)), rng.choice((100, 128, 250))
            descs, p = tuple(cyclic(r, q, nb, nb, 2, 4, c) for r, q in ((m, k), (k, n), (m, n))), 8 * c
        problems.append((descs, p))
    seen = [set() for _ in problems]
    for room in (False, True):                                          # (without room first: buffers taken once stay in a pool)
        for i, (descs, p) in enumerate(problems):
            for aligned in (True, False):
                rec.so.rec_set_limit(2 ** 63 if room else rec.so.rec_live() + (120 << 20))      # tables and partial tiles, no copies
                q = Product(descs, p)
                q.run(q.args(aligned), 0, rec.stream())
                seen[i].add((q.plan.small_tile(), q.plan.ran_k_split()))
                if q.plan.ran_dense():
                    assert room and not q.plan.ran_k_split()
                    dense += 1
                    # (what the plan's own list does where it is asked for by name)
                    own = Product(descs, p, q.b.DMM_MERGE_ALWAYS) if q.plan.num_merged_items() else q
                    own.run(own.args(aligned, 1), 0 if own is not q else q.b.DMM_NO_MERGE, rec.stream())
                    was_cut += own.plan.ran_k_split()
                q.plan.destroy()
    for (descs, _), s in zip(problems, seen):
        assert len(s) == 1, (descs, s)
    cut = sum(split for s in seen for _, split in s)
    assert dense >= 20 and cut >= 8 and was_cut >= 4, (dense, cut, was_cut)


def a_failed_allocation_costs_no_call(rec):
    """One device allocation after another of a call that would run on copies fails, alone or with the one behind
    it: the call then runs its own work list (whose tables there is room for; a copy that was under way by
    then is for nothing), and goes on like that."""
    block, cyclic, keep, s = workloads.block_desc, workloads.block_cyclic_desc, [], rec.stream()
    p = Product(tuple(cyclic(8192, 8192, 128, 128, 2, 4, 1) for _ in range(3)), 8)
    rec.so.rec_fail_allocations(0, 3)
    p.run(p.args(False), 0, s)               # no room for copies
    assert rec.so.rec_failed() and [o[1] for o in rec.launches()] == ["grouped_gemm_comp_kernel"]
    for descs, ranks in ((tuple(cyclic(r, q, 100, 100, 2, 4, 1) for r, q in ((4101, 8200), (8200, 4099), (4101, 4099))), 8),
                         (tuple(cyclic(r, q, 100, 100, 2, 4, 2) for r, q in ((4200, 4099), (4099, 4102), (4200, 4102))), 16),
                         ((block(6656, 3840, 8, 8), block(3840, 5376, 8, 8), block(6656, 5376, 8, 8)), 64)):
        for times in (1, 2):
            n, failed = 0, True
            while failed:
                for _ in range(3):                                       # (plans that live on keep the pools of tables empty)
                    keep.append(Product(descs, ranks))
                    keep[-1].run(keep[-1].args(False, 99), 0, s)
                p = Product(descs, ranks)
                args = p.args(False, n)
                at = len(rec.ops())
                rec.so.rec_fail_allocations(n, times)
                p.run(args, 0, s)
                failed = bool(rec.so.rec_failed())
                rec.so.rec_fail_allocations(-1, 0)
                first = [o[1] for o in rec.launches(at)]
                at = len(rec.ops())
                p.run(args, 0, s)
                again = [o[1] for o in rec.launches(at)]
                assert again == [o for o in first if o != "pack_kernel" or not failed] and p.plan.last_execute().table_reused
                assert ("pack_kernel" in again) == p.plan.ran_dense() == (not failed), (n, again)
                assert len([o for o in first if "gemm" in o]) == 1, first
                rec.check_tables()
                keep.append(p)
                n += 1
            assert n >= 3                    # two sets of tables, none


def calls_can_be_captured(rec):
    """A plan that has run on a stream runs again while that stream is captured (the runtime then refuses waits
    for events that the stream recorded before): on the operands, on copies, with tiles cut along K, and by
    every kind of kernel."""
    block, cyclic = workloads.block_desc, workloads.block_cyclic_desc
    fine = tuple(cyclic(8192, 8192, 128, 128, 2, 4, 1) for _ in range(3))
    long = (block(1024, 16384, 8, 1), block(16384, 1024, 1, 8), block(1024, 1024, 4, 2))
    column = (block(32, 12288, 1, 1, replication=8), block(12288, 49152, 1, 8), block(32, 49152, 1, 8))
    for descs, ranks, kw, kernels in ((row_col(8192, 8192, 8192), 8, {}, ["grouped_gemm_kernel"]),
                                      (fine, 8, {}, ["pack_kernel", "grouped_gemm_comp_kernel"]),
                                      (long, 8, {}, ["small_gemm_kernel", "small_sum_kernel"]),
                                      (column, 8, {}, None),
                                      (row_col(2501, 1999, 1777), 8, dict(dtype="f32"), None)):
        p, s, other = Product(descs, ranks, **kw), rec.stream(), rec.stream()
        args = p.args()
        p.run(args, 0, other)
        p.run(args, 0, s)
        rec.so.rec_set_capturing(s, 1)
        for _ in range(2):
            at = len(rec.ops())
            p.run(args, 0, s)
            got = [o[1] for o in rec.launches(at)]
            assert got == kernels or kernels is None, got
        rec.so.rec_set_capturing(s, 0)
        p.run(args, 0, other)
        p.run(p.args(where=1), 0, s)
        rec.check_tables()


def a_stream_for_every_thread(rec):
    """hipStreamPerThread is another stream in every thread: new tables wait for the calls of all of them, one
    thread's call does not take another's place."""
    per_thread = 2
    p = Product(row_col(1024, 512, 1024), 8)
    args, others = p.args(), p.args(where=1)
    for a in (args, args, args, others):
        t = threading.Thread(target=p.run, args=(a, 0, per_thread))
        t.start()
        t.join()
    assert len({o[2] for o in rec.launches()}) == 4
    rec.check_tables()
    p.plan.destroy()


class Copies:
    """Where the copies of the calls of a scenario lay, and which launches read and wrote them."""

    def __init__(self, rec):
        self.rec, self.calls = rec, []

    def run(self, p, args, stream):
        """A call on copies; the address range of the copies."""
        at = len(self.rec.ops())
        p.run(args, 0, stream)
        launches = self.rec.launches(at)
        assert p.plan.ran_dense() and launches[0][1] == "pack_kernel", launches
        jobs, _, _ = _pack_tables(self.rec, launches[0][0])
        lo = min(j[0] for j in jobs)
        hi = max(j[0] + j[3] * j[1] for j in jobs)
        for first, last, lo2, hi2 in self.calls:
            if lo < hi2 and lo2 < hi:
                assert self.rec.before(last, launches[0][0]), "copies are made over those that an earlier product reads"
        self.calls.append((launches[0][0], launches[-1][0], lo, hi))
        self.rec.check_tables()
        return lo, hi


def copies_share_their_memory(rec):
    """Many plans that are kept, all on copies: on one stream they take one buffer, whose place stays good for
    their tables; on several streams they overlap only in order; all copies together stay within 2 GiB."""
    cyclic = workloads.block_cyclic_desc
    sizes = [(8192, 8192, 8192, 128), (4101, 2051, 4099, 100), (8192, 4096, 8192, 128), (8192, 8192, 8192, 128), (12288, 12288, 8192, 128)]
    plans = []
    for m, k, n, nb in sizes:
        p = Product(tuple(cyclic(r, q, nb, nb, 2, 4, 1) for r, q in ((m, k), (k, n), (m, n))), 8)
        plans.append((p, p.args(False, len(plans))))
    copies, s = Copies(rec), rec.stream()
    start = rec.so.rec_live()
    for times in range(3):
        for p, args in plans[::-1]:
            copies.run(p, args, s)
            assert times < 1 or p.plan.last_execute().table_reused
    assert len({lo for _, _, lo, _ in copies.calls}) == 1
    assert rec.so.rec_live() - start < (520 << 20)
    import random
    rng, streams = random.Random(5), [rec.stream() for _ in range(6)] + [s]
    for _ in range(60):
        p, args = rng.choice(plans)
        copies.run(p, args, rng.choice(streams))
        assert rec.so.rec_live() - start <= (2 << 30) + (64 << 20)
    for p, _ in plans:
        p.plan.destroy()
    big = Product(tuple(cyclic(r, q, 128, 128, 2, 4, 1) for r, q in ((16384, 24576), (24576, 16384), (16384, 16384))), 8)   # 1.6 GB: the others make room
    big.run(big.args(False, 9), 0, s)
    assert big.plan.ran_dense() and rec.so.rec_live() - start <= (2 << 30) + (64 << 20)
    # tables that need more than there is left take it from the copies
    rec.so.rec_set_limit(rec.so.rec_live() + (1 << 16))
    p = Product(tuple(cyclic(4096, 4096, 16, 16, 2, 4, 1) for _ in range(3)), 8)
    p.run(p.args(), 0, s)


def a_captured_call_keeps_its_copies(rec):
    """The buffer of a call that is captured goes to no other plan until its own is destroyed."""
    cyclic = workloads.block_cyclic_desc
    d = tuple(cyclic(8192, 8192, 128, 128, 2, 4, 1) for _ in range(3))
    p, q, r = (Product(d, 8) for _ in range(3))
    copies, s, other = Copies(rec), rec.stream(), rec.stream()
    pa, qa, ra = p.args(False), q.args(False, 1), r.args(False, 2)
    copies.run(p, pa, s)
    where = copies.run(q, qa, s)
    rec.so.rec_set_capturing(s, 1)
    assert copies.run(p, pa, s) == where
    rec.so.rec_set_capturing(s, 0)
    for x, args in ((q, qa), (r, ra), (q, qa)):
        for stream in (s, other):
            lo, hi = copies.run(x, args, stream)
            assert hi <= where[0] or where[1] <= lo
    assert copies.run(p, pa, other) == where
    p.plan.destroy()
    rec.so.rec_set_limit(rec.so.rec_live())
    assert copies.run(Product(d, 8), p.args(False, 3), rec.stream())


def free_memory_does_not_show_in_the_cut(rec):
    """A small product that is cut along K, with less and less room for its partial tiles: the same tiles, cut
    into the same ranges, in more launches; every workgroup runs once."""
    for descs, ranks, dtype in ((row_col(1024, 16384, 1024), 8, "bf16"), (row_col(2501, 1999, 1777), 8, "f32")):
        seen, launches, keep = set(), [], []
        for room in (1 << 40, 40 << 20, 20 << 20, 6 << 20):
            p = Product(descs, ranks, dtype=dtype)
            rec.so.rec_set_limit(rec.so.rec_live() + room)
            at = len(rec.ops())
            p.run(p.args(), 0, rec.stream())
            got = rec.launches(at)
            assert [o[1] for o in got] == ["small_gemm_kernel", "small_sum_kernel"] * (len(got) // 2)
            k = p.plan.last_kernels()
            blocks = [sum(rec.so.rec_blocks(o[0]) for o in got if o[1] == name) for name in ("small_gemm_kernel", "small_sum_kernel")]
            seen.add((k.small_rows, k.small_cols, k.small_runs, *blocks))
            launches.append(len(got))
            rec.check_tables()
            keep.append(p)                           # (nothing goes back to the pools)
        assert len(seen) == 1 and k.small_runs > 1 and launches[0] == 2 < launches[-1] and launches == sorted(launches), (seen, launches)


def an_error_on_one_stream_leaves_the_others_waited_for(rec):
    p = Product(row_col(1024, 512, 1024), 8)
    args, streams = p.args(), [rec.stream() for _ in range(3)]
    for s in streams:
        p.run(args, 0, s)
    readers = [o[0] for o in rec.launches()]
    rec.so.rec_fail_wait(0)
    p.plan.destroy()
    rec.so.hipGetLastError()
    q = Product(row_col(1024, 520, 1024), 8)
    q.run(q.args(), 0, rec.stream())
    mark = rec.ops()[-1][0]
    assert [rec.before(r, mark) for r in readers] == [False, True, True]


def a_copy_whose_product_failed_is_waited_for(rec):
    """The copy is launched before the product's tables are in place; if these fail, the next call's tables
    wait for the copy all the same."""
    cyclic = workloads.block_cyclic_desc
    p = Product(tuple(cyclic(8192, 8192, 128, 128, 2, 4, 1) for _ in range(3)), 8)
    s, other = rec.stream(), rec.stream()
    for i in range(2):
        p.run(p.args(False, i), 0, s)
    at = len(rec.ops())
    rec.so.rec_fail_wait(1)                      # (the third tables reuse the first staging slot: of the copy, of the product)
    try:
        p.run(p.args(False, 2), 0, s)
        raise AssertionError("the wait did not fail")
    except p.b.DmmError:
        rec.so.hipGetLastError()
    assert [o[1] for o in rec.launches(at)] == ["pack_kernel"]
    p.run(p.args(False, 3), 0, other)
    assert p.plan.ran_dense()
    rec.check_tables()
    p.plan.destroy()


def what_was_slower_stays_as_it_is(rec):
    """Products that were timed and found slower on copies run on their operands; batches of 33 to 64 rows do not
    take two tile rows of the 32-row shape, which would stream the weights twice."""
    block = workloads.block_desc
    for descs, ranks, aligned in (((block(11441, 9344, 1, 1, replication=8), block(9344, 4245, 1, 8), block(11441, 4245, 1, 8)), 8, True),):
        p = Product(descs, ranks)
        p.run(p.args(aligned), 0, rec.stream())
        assert not p.plan.ran_dense() and p.plan.small_tile() is None
    for m, k, n in ((48, 4160, 34486), (64, 6115, 48707), (64, 10392, 38990), (64, 15936, 23552), (60, 16187, 10892)):
        p = Product((block(m, k, 1, 1, replication=8), block(k, n, 1, 8), block(m, n, 1, 8)), 8)
        p.run(p.args(), 0, rec.stream())
        assert p.plan.small_tile() in (None, (64, 128)), (m, k, n, p.plan.small_tile())
    # operands from memory in little more than one workgroup per CU; a second launch that takes longer than it saves; long K
    # at odd places in 128 x 128 tiles
    for m, k, n in ((43, 13723, 16385), (40, 10240, 11088), (8, 14848, 16652), (112, 13312, 33360)):
        p = Product((block(m, k, 1, 1, replication=8), block(k, n, 1, 8), block(m, n, 1, 8)), 8)
        at = len(rec.ops())
        p.run(p.args(), p.b.DMM_C_BF16, rec.stream())
        if p.plan.small_tile():
            wgs = max(rec.so.rec_blocks(o[0]) for o in rec.launches(at) if o[1] == "small_gemm_kernel")
            assert not (256 < wgs < 340 or 512 < wgs < 600), (m, k, n, wgs)
    for d in (tuple(block(r, c, 4, 2) for r, c in ((640, 384), (384, 832), (640, 832))), row_col(256, 896, 321)):
        p = Product(d, 8)
        p.run(p.args(), 0, rec.stream())
        assert p.plan.small_tile() and p.plan.last_kernels().small_runs == 1, (d, p.plan.last_kernels().small_runs)
    p = Product((block(82, 2944, 1, 1, replication=8), block(2944, 33024, 1, 8), block(82, 33024, 1, 8)), 8)
    p.run(p.args(), p.b.DMM_C_BF16, rec.stream())
    assert p.plan.small_tile() == (128, 128) and p.plan.last_kernels().small_runs == 1      # (B fits the last-level cache)
    p = Product(uneven(4985, 9842, 3072, 286), 15)
    p.run(p.args(False), 0, rec.stream())
    assert p.plan.small_tile() is None


def copies_do_not_lie_across_a_4gb_line(rec):
    """The merged macro-tile kernel loads a K-segment step by step that a multiple of 2^32 runs through."""
    cyclic = workloads.block_cyclic_desc
    d = tuple(cyclic(8192, 8192, 128, 128, 2, 4, 1) for _ in range(3))
    for limit in (None, 300 << 20):                              # with and without room for two buffers at a time
        line = (0x7100 if limit else 0x7000) << 32
        rec.so.rec_next_at(line - (48 << 20))
        if limit:
            rec.so.rec_set_limit(rec.so.rec_live() + limit)
        p, copies = Product(d, 8), Copies(rec)
        lo, hi = copies.run(p, p.args(False), rec.stream())
        assert (lo >> 32 == (hi - 1) >> 32) == (limit is None)
        rec.so.rec_set_limit(2 ** 63)


def _small_tables(rec, start=0):
    """The tables that a kernel on the caller's stream wrote."""
    return [o for o in rec.ops(start) if o[1] == "copy" and rec.so.rec_more(o[0], 0) == 1]


def a_table_whose_call_failed_is_not_written_late(rec):
    """A table is written on the caller's stream, then the call's launch fails.  The next call's table, copied on the
    library's own stream (its caller's is being captured), comes behind it."""
    p = Product(tuple(workloads.block_desc(256, 256, 2, 2) for _ in range(3)), 4, dtype="f32")
    s, other = rec.stream(), rec.stream()
    for i, streams in enumerate(((s, s), (s, other), (other, s))):
        at = len(rec.ops())
        rec.so.rec_fail_launches(1)
        try:
            p.run(p.args(where=3 * i), 0, streams[0])
            raise AssertionError("the call did not fail")
        except p.b.DmmError:
            rec.so.rec_fail_launches(0)
        assert len(_small_tables(rec, at)) == 1 and not rec.launches(at)
        rec.so.rec_set_capturing(streams[1], 1)
        p.run(p.args(where=3 * i + 1), 0, streams[1])
        rec.so.rec_set_capturing(streams[1], 0)
        assert len(_small_tables(rec, at)) == 1 and len(rec.launches(at)) == 1
        rec.check_tables()
        p.run(p.args(where=3 * i + 2), 0, streams[0])
        assert len(_small_tables(rec, at)) == 2
        rec.check_tables()


def a_buffer_given_up_for_a_larger_one_is_not_written_late(rec):
    """A table is copied, then the call's launch fails; the next call needs a larger buffer.  The plan that takes the
    smaller one over writes its table behind that copy."""
    block, s = workloads.block_desc, [rec.stream() for _ in range(3)]
    p = Product((block(512, 1024, 16, 16), block(1024, 512, 1, 8), block(512, 512, 1, 8)), 256)
    rec.so.rec_fail_launches(1)
    try:
        p.run(p.args(), 0, s[0])
        raise AssertionError("the call did not fail")
    except p.b.DmmError:
        rec.so.rec_fail_launches(0)
    late = rec.ops()[-2]
    assert late[1] == "copy" and late[4] < 65536 and not _small_tables(rec) and not rec.launches()
    p.run(p.args(), p.b.DMM_NO_MERGE, s[1])
    assert max(o[4] for o in rec.ops() if o[1] == "copy") > 65536
    q = Product(tuple(block(256, 256, 2, 2) for _ in range(3)), 4, dtype="f32")
    q.run(q.args(), 0, s[2])
    assert [o[3] for o in _small_tables(rec)] == [late[3]]       # the same buffer
    rec.check_tables()


def events_are_recorded_between_launches(rec):
    """Launches record the events that stand for their calls; in a long row of calls, on a plan that is kept or on new ones,
    an event is recorded by a call of its own now and then, so that the runtime lets go of the launches before."""
    d = tuple(workloads.block_desc(256, 256, 2, 2) for _ in range(3))
    s = rec.stream()
    p = Product(d, 4, dtype="f32")
    args = p.args()
    for new in (False, True):
        at = len(rec.ops())
        for _ in range(256):
            q = Product(d, 4, dtype="f32") if new else p
            q.run(args, 0, s)
        row = [o[1] for o in rec.ops(at) if o[2] == s and o[1] in ("event", "small_gemm_kernel")]
        assert row.count("small_gemm_kernel") == 256 and row.count("event") <= 16
        while "event" in row:
            assert row.index("event") <= 64
            row = row[row.index("event") + 1:]
        assert len(row) <= 64
    rec.check_tables()


def small_tables_travel_with_a_kernel(rec):
    """Tables of up to 3584 bytes, whatever the number of cuts in them; larger ones, and under capture all, are copied."""
    block, s = workloads.block_desc, rec.stream()
    sizes = set()
    for descs, ranks, dtype in ((row_col(256, 256, 256, 4), 4, "f32"), (row_col(2048, 1024, 2048, 8), 8, "bf16"),
                                (tuple(block(300, 300, 1, 1) for _ in range(3)), 1, "bf16"), (tuple(block(300, 300, 2, 2) for _ in range(3)), 4, "f32"),
                                ((block(300, 700, 1, 7), block(700, 300, 5, 1), block(300, 300, 2, 3)), 7, "f32"),
                                ((block(300, 6000, 1, 50), block(6000, 300, 40, 1), block(300, 300, 2, 3)), 50, "f32")):
        for capture in (0, 1):
            p, at = Product(descs, ranks, dtype=dtype), len(rec.ops())
            rec.so.rec_set_capturing(s, capture)
            p.run(p.args(where=1 + capture), 0, s)
            rec.so.rec_set_capturing(s, 0)
            assert p.plan.small_tile()
            written = [o for o in rec.ops(at) if o[1] == "copy"]
            assert len(written) == 1 and written[0][4] % 8 == 0
            assert len(_small_tables(rec, at)) == (0 if capture else int(written[0][4] <= 3584))
            sizes.add(written[0][4] <= 3584)
            rec.check_tables()
    assert sizes == {True, False}


def handles_that_name_a_stream(rec):
    """hipStreamLegacy and hipStreamPerThread: launches that record events are not made on these; the null stream and the
    former are one."""
    d = tuple(workloads.block_desc(256, 256, 2, 2) for _ in range(3))
    long = (workloads.block_desc(1024, 16384, 8, 1), workloads.block_desc(16384, 1024, 1, 8), workloads.block_desc(1024, 1024, 4, 2))
    for descs, ranks, dtype in ((d, 4, "f32"), (long, 8, "bf16")):
        p = Product(descs, ranks, dtype=dtype)
        for i, stream in enumerate((0, 1, 2, 0, rec.stream(), 2, 1)):
            for _ in range(2):
                at = len(rec.ops())
                p.run(p.args(where=i % 3), 0, stream)
                own = [o[1] for o in rec.ops(at) if o[2] == rec.ops()[-1][2]]
                assert stream not in (1, 2) or own[-1] == "event"
        rec.check_tables()
        p.plan.destroy()


SCENARIOS = [dense_calls_and_others_on_two_streams, destroy_waits_for_every_stream, scratch_is_not_shared_by_calls_that_overlap,
             more_streams_than_the_plan_remembers, reports_say_what_ran,
             the_copies_hold_the_k_steps_of_the_operands, copies_do_not_show_in_the_bits, a_failed_allocation_costs_no_call,
             calls_can_be_captured, a_stream_for_every_thread,
             copies_share_their_memory, a_captured_call_keeps_its_copies,
             free_memory_does_not_show_in_the_cut,
             an_error_on_one_stream_leaves_the_others_waited_for,
             a_copy_whose_product_failed_is_waited_for, what_was_slower_stays_as_it_is,
             copies_do_not_lie_across_a_4gb_line, a_table_whose_call_failed_is_not_written_late,
             a_buffer_given_up_for_a_larger_one_is_not_written_late, events_are_recorded_between_launches,
             small_tables_travel_with_a_kernel, handles_that_name_a_stream]


# ---- the tests ----------------------------------------------------------------------------------------

@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    so = str(tmp_path_factory.mktemp("recorder") / "hip_recorder.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(ROOT, "tests", "native", "hip_recorder.cpp"), "-o", so], check=True, capture_output=True, text=True)
    return so


@pytest.mark.parametrize("scenario", [f.__name__ for f in SCENARIOS])
def test_scenario(recorder, scenario):
    run = subprocess.run([sys.executable, os.path.abspath(__file__), recorder, scenario], capture_output=True, text=True,
                         cwd=ROOT, timeout=300)
    assert run.returncode == 0, run.stdout[-2000:] + run.stderr[-4000:]


if __name__ == "__main__":
    {f.__name__: f for f in SCENARIOS}[sys.argv[2]](Recorder(sys.argv[1]))
