"""GPU tests of the symmetric heap, translation (device vs host twin), the
atomic and value (load/store) verbs of the device API, and the heap tile
copy (bit-exact vs oracle)."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import workload
from tests.gpu_util import require_gpu, sym

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()
    yield
    torch.cuda.synchronize()


# ---------------------------------------------------------------- heap + translation

def test_library_owned_heap_geometry_and_errors():
    pkg = sym()
    h = pkg.symtile_heap_create(0, 8, 3 << 20)          # 3 MiB -> 4 MiB stride
    try:
        w, stride, used, dev = pkg.symtile_heap_info(h)
        assert (w, stride, used, dev) == (8, 4 << 20, 0, 0)
        dev_bases, host = pkg.symtile_heap_bases(h)
        assert dev_bases and all(host[r] - host[0] == r * stride for r in range(8))
        assert host[0] % 256 == 0
        o1 = pkg.symtile_heap_alloc(h, 100, 0)
        o2 = pkg.symtile_heap_alloc(h, 10, 4096)
        assert o1 == 0 and o2 == 4096
        assert pkg.symtile_heap_ptr(h, 5, o2) == host[5] + 4096
        with pytest.raises(pkg.SymtileError) as e:
            pkg.symtile_heap_alloc(h, stride, 0)
        assert e.value.name == "ENOMEM"
        with pytest.raises(pkg.SymtileError) as e:
            pkg.symtile_heap_alloc(h, 16, 3)
        assert e.value.name == "EINVAL"
        # the device bases array holds the same addresses
        got = (ctypes.c_uint64 * 8)()
        t = torch.empty(8, dtype=torch.int64, device="cuda")
        hip = ctypes.CDLL("libamdhip64.so")
        hip.hipMemcpy.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int]
        assert hip.hipMemcpy(ctypes.addressof(got), ctypes.c_void_p(dev_bases), 64, 2) == 0
        assert list(got) == host
        del t
        pkg.symtile_barrier(h, 0)
    finally:
        pkg.symtile_heap_destroy(h)
    with pytest.raises(pkg.SymtileError):
        pkg.symtile_heap_create(0, 9, 1 << 20)
    with pytest.raises(pkg.SymtileError):
        pkg.symtile_heap_create(0, 2, 0)


def test_translation_host_twin_invariants():
    pkg = sym()
    heap = pkg.Heap(4, 1 << 21)
    h = heap.handle
    _, host = heap.bases()
    rng = np.random.default_rng(0)
    for _ in range(50):
        a, b = rng.integers(0, 4, size=2)
        off = int(rng.integers(0, heap.stride))
        p = host[a] + off
        q = pkg.symtile_translate(h, p, int(a), int(b))
        assert q - host[b] == off                                  # offset preserved
        assert pkg.symtile_translate(h, q, int(b), int(a)) == p    # round trip
        assert pkg.symtile_translate(h, p, int(a), int(a)) == p    # identity
    for bad_p, a in ((host[1], 0), (host[0] - 1, 0), (host[3] + heap.stride, 3)):
        with pytest.raises(pkg.SymtileError) as e:
            pkg.symtile_translate(h, bad_p, a, 1)
        assert e.value.name == "EINVAL"
    with pytest.raises(pkg.SymtileError):
        pkg.symtile_translate(h, host[0], 0, 4)


def test_translation_device_matches_host_twin():
    pkg = sym()
    heap = pkg.Heap(8, 1 << 21)
    _, host = heap.bases()
    rng = np.random.default_rng(1)
    n = 1000
    for a, b in ((0, 7), (3, 1), (5, 5), (7, 0)):
        offs = rng.integers(0, heap.stride, size=n)
        ins = torch.tensor([host[a] + int(o) for o in offs], dtype=torch.int64, device="cuda")
        outs = torch.zeros_like(ins)
        pkg.symtile_translate_device(heap.handle, ins.data_ptr(), n, a, b, outs.data_ptr(),
                                     pkg.current_stream())
        heap.barrier()
        want = [pkg.symtile_translate(heap.handle, host[a] + int(o), a, b) for o in offs]
        assert outs.cpu().numpy().astype(np.uint64).tolist() == want


def test_fill_and_views_alias_the_slots():
    pkg = sym()
    heap = pkg.Heap(3, 1 << 20)
    off = heap.alloc(4096)
    heap.fill(-1, off, 4096, 0xAB)
    heap.fill(1, off + 16, 32, 0x01)
    heap.fill(2, off + 3, 5, 0x7F)                     # unaligned path
    torch.cuda.synchronize()
    v = heap.slots_view(off, (4096,), torch.uint8).cpu().numpy()
    assert np.all(v[0] == 0xAB)
    assert np.all(v[1][16:48] == 1) and np.all(v[1][:16] == 0xAB) and np.all(v[1][48:] == 0xAB)
    assert np.all(v[2][3:8] == 0x7F) and v[2][2] == 0xAB and v[2][8] == 0xAB
    with pytest.raises(pkg.SymtileError):
        heap.fill(0, heap.stride - 8, 16, 0)


# ---------------------------------------------------------------- atomics (device API)

def _atomic(pkg, heap, op, sem, scope, n, operand, init, compare=0, frm=1, to=5):
    off = heap.alloc(256)
    heap.slots_view(off, (64,), torch.int32).zero_()
    heap.view(to, off, (1,), torch.int32).fill_(init)
    old = torch.zeros(n, dtype=torch.int32, device="cuda")
    pkg.symtile_atomic_exercise(heap.handle, pkg.ATOMIC_OPS[op], pkg.SEMS[sem], pkg.SCOPES[scope],
                                off, frm, to, n, operand, compare, old.data_ptr(),
                                pkg.current_stream())
    heap.barrier()
    words = heap.slots_view(off, (64,), torch.int32).cpu().numpy().view(np.uint32)
    others = [s for s in range(heap.world) if s != to]
    assert np.all(words[others] == 0), "atomic touched another slot"
    assert np.all(words[to][1:] == 0)
    return int(words[to][0]), old.cpu().numpy().view(np.uint32)


def _fold(fn, init, vals):
    acc = init
    for v in vals:
        acc = fn(acc, v) & 0xFFFFFFFF
    return acc


# verb -> (operand, initial word, compare) of the exercise; thread t applies operand + t
_VERB_ARGS = {"add": (1, 7, 0), "xchg": (1000, 5, 0), "cas": (100, 9, 9),
              "and": (0xFFFFFFF0, 0xFF, 0), "or": (0x100, 0, 0), "xor": (3, 0x55, 0),
              "min": (50, 200, 0), "max": (50, 200, 0)}


@pytest.mark.parametrize("op", list(_VERB_ARGS))
@pytest.mark.parametrize("sem", ["relaxed", "acquire", "release", "acq_rel"])
@pytest.mark.parametrize("scope", ["block", "gpu", "sys"])
def test_atomic_verb_results_every_order_and_scope(op, sem, scope):
    """Every atomic verb of the device API under all 12 ordering x scope
    pairs (Section 3.3.3): n threads of several workgroups apply it to one
    word of another rank's slot through a translated address; the final word
    and the values the threads observed follow from the verb alone (whatever
    order the threads ran in), and no other word of any slot changes."""
    pkg = sym()
    heap = pkg.Heap(8, 1 << 21)
    n = 300 if op != "and" else 4
    operand, init, compare = _VERB_ARGS[op]
    vals = [(operand + t) & 0xFFFFFFFF for t in range(n)]
    final, old = _atomic(pkg, heap, op, sem, scope, n, operand, init, compare=compare)
    if op == "add":
        # every addend is positive, so the observed values are distinct
        assert final == (init + sum(vals)) % 2 ** 32
        assert len(np.unique(old)) == n
    elif op == "xchg":
        assert set(old.tolist()) | {final} == set(vals) | {init}     # a permutation chain
        assert len(np.unique(old)) == n
    elif op == "cas":
        assert final in vals and int(np.sum(old == init)) == 1       # exactly one winner
        assert np.all((old == init) | (old == final))
    else:
        fn = {"and": lambda a, b: a & b, "or": lambda a, b: a | b, "xor": lambda a, b: a ^ b,
              "min": min, "max": max}[op]
        assert final == _fold(fn, init, vals)


# ---------------------------------------------------------------- value verbs (device API)

def _value_heap(pkg, world, nbytes, seed):
    """Heap with every slot filled with seeded random bytes; returns the
    heap, the region offsets and the host copy of every slot before the call."""
    heap = pkg.Heap(world, 3 * nbytes + 4096)
    src, dst = heap.alloc(nbytes + 64, 256), heap.alloc(nbytes + 64, 256)
    g = torch.Generator().manual_seed(seed)
    span = dst + nbytes + 64
    before = torch.randint(0, 256, (world, span), generator=g, dtype=torch.uint8)
    heap.slots_view(0, (span,), torch.uint8).copy_(before.cuda())
    return heap, src, dst, before.numpy(), span


@pytest.mark.parametrize("op", ["load", "store"])
@pytest.mark.parametrize("nbytes,nt", [(16, 0), (4096, 1), (3 * 4096 * 256 + 48, 0),
                                       (16 * 4096 * 256 + 16 * 77, 1)])
def test_value_verbs_move_bitwise_copies(op, nbytes, nt):
    pkg = sym()
    world, cur, remote = 5, 1, 3
    heap, src, dst, before, span = _value_heap(pkg, world, nbytes, seed=nbytes + nt)
    pkg.symtile_value_exercise(heap.handle, pkg.LOAD if op == "load" else pkg.STORE, src, dst,
                               nbytes, cur, remote, nt, pkg.current_stream())
    heap.barrier()
    after = heap.slots_view(0, (span,), torch.uint8).cpu().numpy()
    want = before.copy()
    # load: remote's source lands in cur's destination; store: the reverse
    rd, wr = (remote, cur) if op == "load" else (cur, remote)
    want[wr, dst:dst + nbytes] = before[rd, src:src + nbytes]
    assert np.array_equal(after, want)


def test_value_verbs_same_slot_and_empty():
    pkg = sym()
    heap, src, dst, before, span = _value_heap(pkg, 2, 1024, seed=3)
    pkg.symtile_value_exercise(heap.handle, pkg.STORE, src, dst, 1024, 0, 0, 0,
                               pkg.current_stream())
    pkg.symtile_value_exercise(heap.handle, pkg.LOAD, src, dst, 0, 1, 0, 0,
                               pkg.current_stream())
    heap.barrier()
    after = heap.slots_view(0, (span,), torch.uint8).cpu().numpy()
    want = before.copy()
    want[0, dst:dst + 1024] = before[0, src:src + 1024]
    assert np.array_equal(after, want)


def test_value_verbs_reject_bad_arguments():
    pkg = sym()
    heap = pkg.Heap(4, 1 << 20)
    off = heap.alloc(1 << 16)
    st = pkg.current_stream()
    good = dict(op=pkg.LOAD, src=off, dst=off + 4096, n=1024, cur=0, remote=2, nt=0)
    bad = [dict(op=2), dict(src=off + 8), dict(dst=off + 4100), dict(n=1000), dict(cur=4),
           dict(remote=-1), dict(nt=2), dict(dst=heap.stride - 512),
           dict(src=heap.stride + 16), dict(remote=0, dst=off + 512)]
    for change in bad:
        a = {**good, **change}
        with pytest.raises(pkg.SymtileError) as e:
            pkg.symtile_value_exercise(heap.handle, a["op"], a["src"], a["dst"], a["n"],
                                       a["cur"], a["remote"], a["nt"], st)
        assert e.value.name == "EINVAL", change
    heap.barrier()


# ---------------------------------------------------------------- heap tile copy

def _copy_heap(pkg, world, rows, cols, dtype_t):
    esize = torch.empty((), dtype=dtype_t).element_size()
    nbytes = rows * cols * esize
    heap = pkg.Heap(world, 2 * nbytes + (1 << 20))
    src = heap.alloc(nbytes)
    dst = heap.alloc(nbytes)
    flags = heap.alloc(1 << 16)
    return heap, src, dst, flags


@pytest.mark.parametrize("mode", [0, 1], ids=["put", "get"])
@pytest.mark.parametrize("tile,per_wg", [(64, 0), (128, 0), (256, 0), (128, 1), (64, 7), (64, 96)])
def test_heap_tile_copy_workload_bitexact(tile, per_wg, mode):
    """All 8 ranks copy send -> recv of rank (r+1) mod 8, 2048 x 2048 fp32
    (put: each rank writes the next rank's heap; get: each rank reads the
    previous rank's heap)."""
    pkg = sym()
    wl = workload.HEAP_COPY
    heap, src, dst, flags = _copy_heap(pkg, wl.world, wl.rows, wl.cols, torch.float32)
    send = workload.copy_send(wl, seed=0)
    heap.slots_view(src, (wl.rows, wl.cols), torch.float32).copy_(send.cuda())
    heap.slots_view(dst, (wl.rows, wl.cols), torch.int32).fill_(-1)
    pkg.symtile_tile_copy(heap.handle, src, dst, wl.rows, wl.cols, wl.cols, pkg.F32, tile, tile,
                          wl.shift, -1, flags, tiles_per_wg=per_wg, stream=pkg.current_stream(),
                          mode=mode)
    heap.barrier()
    recv = heap.slots_view(dst, (wl.rows, wl.cols), torch.float32).cpu().numpy()
    ntiles = (wl.rows // tile) * (wl.cols // tile)
    fl = heap.slots_view(flags, (ntiles,), torch.int32).cpu().numpy()
    want, want_flags = oracle.tile_copy(send.numpy(), np.full_like(send.numpy(), np.nan),
                                        tile, tile, wl.shift, get=bool(mode))
    assert np.array_equal(recv.view(np.uint32), want.view(np.uint32))
    assert np.array_equal(fl, want_flags.astype(np.int32))


@pytest.mark.parametrize("tile", [64, 128, 256])
def test_heap_tile_copy_timed_matches_untimed(tile):
    """symtile_tile_copy_timed leaves the same heap as symtile_tile_copy (the
    oracle's ring copy, every counter at 1 after one call, at 2 after the
    second) and reports a positive kernel duration; an empty copy reports 0."""
    pkg = sym()
    wl = workload.HEAP_COPY
    heap, src, dst, flags = _copy_heap(pkg, wl.world, wl.rows, wl.cols, torch.float32)
    send = workload.copy_send(wl, seed=3)
    heap.slots_view(src, (wl.rows, wl.cols), torch.float32).copy_(send.cuda())
    heap.slots_view(dst, (wl.rows, wl.cols), torch.int32).fill_(-1)
    ms = pkg.symtile_tile_copy_timed(heap.handle, src, dst, wl.rows, wl.cols, wl.cols, pkg.F32,
                                     tile, tile, wl.shift, -1, flags,
                                     stream=pkg.current_stream())
    assert 0.0 < ms < 100.0
    pkg.symtile_tile_copy(heap.handle, src, dst, wl.rows, wl.cols, wl.cols, pkg.F32, tile, tile,
                          wl.shift, -1, flags, stream=pkg.current_stream())
    heap.barrier()
    recv = heap.slots_view(dst, (wl.rows, wl.cols), torch.float32).cpu().numpy()
    ntiles = (wl.rows // tile) * (wl.cols // tile)
    fl = heap.slots_view(flags, (ntiles,), torch.int32).cpu().numpy()
    want, want_flags = oracle.tile_copy(send.numpy(), np.full_like(send.numpy(), np.nan),
                                        tile, tile, wl.shift)
    assert np.array_equal(recv.view(np.uint32), want.view(np.uint32))
    assert np.array_equal(fl, 2 * want_flags.astype(np.int32))
    assert pkg.symtile_tile_copy_timed(heap.handle, src, dst, 0, wl.cols, wl.cols, pkg.F32,
                                       tile, tile, 1, -1, flags) == 0.0
    heap.barrier()


@pytest.mark.parametrize("mode", [0, 1], ids=["put", "get"])
@pytest.mark.parametrize("case", [(5, 100, 72, 32, 24, 3, "bf16"), (3, 33, 20, 16, 8, 1, "f32"),
                                  (8, 64, 64, 64, 64, 7, "f16")])
def test_heap_tile_copy_ragged_and_single_rank(case, mode):
    pkg = sym()
    world, rows, cols, tr, tc, shift, dt = case
    tdt = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}[dt]
    code = {"bf16": pkg.BF16, "f16": pkg.F16, "f32": pkg.F32}[dt]
    ival = torch.int16 if dt != "f32" else torch.int32
    heap, src, dst, flags = _copy_heap(pkg, world, rows, cols, tdt)
    g = torch.Generator().manual_seed(3)
    send = torch.randint(-2 ** 15, 2 ** 15, (world, rows, cols), generator=g).to(ival)
    heap.slots_view(src, (rows, cols), ival).copy_(send.cuda())
    heap.slots_view(dst, (rows, cols), ival).zero_()
    ntiles = -(-rows // tr) * -(-cols // tc)
    for only in (world - 1, -1):
        heap.slots_view(flags, (ntiles,), torch.int32).zero_()
        heap.slots_view(dst, (rows, cols), ival).zero_()
        pkg.symtile_tile_copy(heap.handle, src, dst, rows, cols, cols, code, tr, tc, shift,
                              only, flags, tiles_per_wg=3, stream=pkg.current_stream(),
                              mode=mode)
        heap.barrier()
        recv = heap.slots_view(dst, (rows, cols), ival).cpu().numpy()
        fl = heap.slots_view(flags, (ntiles,), torch.int32).cpu().numpy()
        want, wf = oracle.tile_copy(send.numpy(), np.zeros_like(send.numpy()), tr, tc, shift,
                                    only_rank=only, get=bool(mode))
        assert np.array_equal(recv, want), only
        assert np.array_equal(fl, wf.astype(np.int32)), only


def test_heap_tile_copy_rejects_bad_arguments():
    pkg = sym()
    heap, src, dst, flags = _copy_heap(pkg, 2, 64, 64, torch.float32)
    h, s = heap.handle, pkg.current_stream()
    bad = [
        (src, dst, 64, 63, 64, pkg.F32, 16, 16, 1, -1, flags),     # cols*4 not 16-B multiple
        (src, src + 64, 64, 64, 64, pkg.F32, 16, 16, 1, -1, flags),  # overlap
        (src + 4, dst, 64, 64, 64, pkg.F32, 16, 16, 1, -1, flags),  # misaligned
        (src, dst, 64, 64, 64, 9, 16, 16, 1, -1, flags),           # dtype
        (src, dst, 64, 64, 64, pkg.F32, 16, 16, 1, 2, flags),      # only_rank out of range
        (src, dst, 64, 64, 64, pkg.F32, 16, 16, 1, -1, src),       # flags overlap data
        # one row with a 512 MiB stride: the out-of-range passes of a tile's
        # last batch would wrap a 32-bit buffer offset
        (src, dst, 1, 64, 1 << 27, pkg.F32, 1, 64, 1, -1, flags),
    ]
    with pytest.raises(pkg.SymtileError) as e:
        pkg.symtile_tile_copy(h, src, dst, 64, 64, 64, pkg.F32, 16, 16, 1, -1, flags, -1, s)
    assert e.value.name == "EINVAL"
    for args in bad:
        with pytest.raises(pkg.SymtileError) as e:
            pkg.symtile_tile_copy(h, *args, 0, s)
        assert e.value.name == "EINVAL", args
    with pytest.raises(pkg.SymtileError) as e:                  # unknown direction
        pkg.symtile_tile_copy(h, src, dst, 64, 64, 64, pkg.F32, 16, 16, 1, -1, flags, 0, s,
                              mode=2)
    assert e.value.name == "EINVAL"
    heap.barrier()


# ---------------------------------------------------------------- memory-model litmus

def _litmus(pkg, heap, pairs, rounds, words, form, scope="gpu", spin_limit=0):
    """Run the message-passing litmus; returns (stale words, rounds checked,
    whether the barrier reported a timeout)."""
    data = heap.alloc(pairs * words * 4)
    flags = heap.alloc(pairs * 8)               # fresh, zeroed counters
    result = torch.zeros(2, dtype=torch.int32, device="cuda")
    pkg.symtile_litmus_mp(heap.handle, data, flags, pairs, rounds, words, pkg.MP_FORMS[form],
                          pkg.SCOPES[scope], spin_limit, result.data_ptr(), pkg.current_stream())
    timed_out = False
    try:
        heap.barrier()
    except pkg.SymtileError as e:
        assert e.name == "ETIMEOUT", e
        timed_out = True
    bad, done = (int(x) for x in result.cpu())
    return bad, done, timed_out


@pytest.mark.parametrize("form", ["fences", "rmw", "cas"])
@pytest.mark.parametrize("scope", ["gpu", "sys"])
def test_litmus_message_passing_release_acquire_sees_every_word(form, scope):
    """Writer -> reader message passing across XCDs (Section 3.3.3), with the
    release/acquire pair at agent (gpu) or system scope carried by separate
    fences, by the read-modify-writes themselves (fetch_add), or by the CAS
    lock handshake: no reader ever sees a word of an older round, and every
    round completes."""
    pkg = sym()
    heap = pkg.Heap(8, 16 << 20)
    bad, done, timed_out = _litmus(pkg, heap, 32, 300, 2048, form, scope)
    assert not timed_out
    assert done == 32 * 300
    assert bad == 0


@pytest.mark.parametrize("scope", ["gpu", "sys"])
def test_litmus_write_through_release_sees_every_word(scope):
    """The kernels' publication of write-through data: the writer stores the
    round write-through, waits for the stores' acknowledgement and adds to
    the counter with no L2 write-back; the reader polls and acquires.  No
    reader on another XCD ever sees a word of an older round."""
    pkg = sym()
    heap = pkg.Heap(8, 16 << 20)
    bad, done, timed_out = _litmus(pkg, heap, 32, 300, 2048, "wt", scope)
    assert not timed_out
    assert done == 32 * 300
    assert bad == 0


@pytest.mark.parametrize("scope", ["gpu", "sys"])
def test_litmus_coherent_reads_without_invalidate_see_every_word(scope):
    """Write-through publication read back with coherent loads: the reader
    polls the counter and reads the round with coherent (sc0 sc1) loads, with
    no acquire fence; no reader ever sees a word of an older round."""
    pkg = sym()
    heap = pkg.Heap(8, 16 << 20)
    bad, done, timed_out = _litmus(pkg, heap, 32, 300, 2048, "wt_coherent", scope)
    assert not timed_out
    assert done == 32 * 300
    assert bad == 0


def test_litmus_plain_reads_without_invalidate_are_reported():
    """The control of the coherent-read form: ordinary loads with no acquire
    fence may hit the reader's own L2 copy of an older round.  No guarantee;
    every round must complete, and the stale-word count is reported."""
    pkg = sym()
    heap = pkg.Heap(8, 16 << 20)
    bad, done, timed_out = _litmus(pkg, heap, 32, 300, 2048, "wt_plain")
    assert not timed_out and done == 32 * 300
    print(f"write-through data read with ordinary loads, no acquire: {bad} stale words of "
          f"{32 * 300 * 2048}")


def test_litmus_ack_only_release_of_write_back_stores_is_reported():
    """The control of the write-through form: the same acknowledgement-only
    release after ordinary (write-back) stores, which may still sit dirty in
    the writer's L2.  No guarantee; the test requires that every round
    completes and reports the stale-word count."""
    pkg = sym()
    heap = pkg.Heap(8, 16 << 20)
    bad, done, timed_out = _litmus(pkg, heap, 32, 300, 2048, "ack")
    assert not timed_out and done == 32 * 300
    print(f"acknowledgement-only release of write-back stores: {bad} stale words of "
          f"{32 * 300 * 2048}")


def test_litmus_relaxed_form_terminates():
    """Without release and acquire the protocol gives no guarantee; the test
    only requires that every round completes (the stale-word count is
    reported)."""
    pkg = sym()
    heap = pkg.Heap(8, 16 << 20)
    bad, done, timed_out = _litmus(pkg, heap, 32, 300, 2048, "relaxed")
    assert not timed_out and done == 32 * 300
    print(f"relaxed message passing: {bad} stale words of {32 * 300 * 2048}")


@pytest.mark.parametrize("form", ["fences", "rmw", "cas"])
def test_litmus_workgroup_scope_across_xcds_is_reported(form):
    """Release/acquire at workgroup (block) scope between workgroups on
    different XCDs: the scope does not cover the other XCD's L2, so the
    protocol gives no guarantee.  The probe is bounded (a short spin limit;
    a pair whose counter never becomes visible times out and stops); the
    test requires only that it ends and reports what it saw."""
    pkg = sym()
    heap = pkg.Heap(8, 16 << 20)
    bad, done, timed_out = _litmus(pkg, heap, 32, 100, 2048, form, "block", spin_limit=1 << 14)
    assert 0 <= done <= 32 * 100
    assert timed_out or done == 32 * 100
    print(f"block-scope {form} message passing across XCDs: {bad} stale words in {done} "
          f"rounds checked of {32 * 100}; timed out: {timed_out}")


def _sb(pkg, heap, pairs, rounds, form, scope):
    off = heap.alloc(pairs * rounds * 16)      # fresh, zeroed words
    out = torch.full((pairs, rounds, 2), -1, dtype=torch.int32, device="cuda")
    pkg.symtile_litmus_sb(heap.handle, off, pairs, rounds, pkg.SB_FORMS[form], pkg.SCOPES[scope],
                          0, out.data_ptr(), pkg.current_stream())
    heap.barrier()
    o = out.cpu().numpy()
    assert np.all((o == 0) | (o == 1)), "a round was not run or an impossible value was read"
    return {(a, b): int(np.sum((o[..., 0] == a) & (o[..., 1] == b))) for a in (0, 1)
            for b in (0, 1)}


@pytest.mark.parametrize("form", ["acq_rel", "seq_cst"])
@pytest.mark.parametrize("scope", ["gpu", "sys"])
def test_litmus_store_buffering_forbidden_outcome_never_seen(form, scope):
    """Store buffering between two threads on different XCDs (Section 3.3.3):
    with acq_rel read-modify-writes, or seq_cst accesses, at agent or system
    scope, the outcome where both threads read 0 never occurs."""
    pkg = sym()
    heap = pkg.Heap(8, 8 << 20)
    hist = _sb(pkg, heap, 64, 2000, form, scope)
    assert sum(hist.values()) == 64 * 2000
    assert hist[(0, 0)] == 0, hist


def test_litmus_store_buffering_relaxed_is_reported():
    """Relaxed stores and loads give no guarantee; the histogram of outcomes
    is reported (both reading 0 is allowed)."""
    pkg = sym()
    heap = pkg.Heap(8, 8 << 20)
    hist = _sb(pkg, heap, 64, 2000, "relaxed", "gpu")
    assert sum(hist.values()) == 64 * 2000
    print(f"relaxed store buffering (r0, r1): {hist}")


def test_litmus_rejects_bad_arguments():
    pkg = sym()
    heap = pkg.Heap(2, 1 << 20)
    data, flags = heap.alloc(4096), heap.alloc(64)
    res = torch.zeros(2, dtype=torch.int32, device="cuda")
    for args, name in (((data, flags, 0, 1, 16, 1, 1), "EINVAL"),       # no pairs
                       ((data, data, 1, 1, 16, 1, 1), "EINVAL"),        # flags overlap data
                       ((data, flags, 1, 1, 16, 8, 1), "EINVAL"),       # unknown form
                       ((data, flags, 1, 1, 16, 1, 3), "EINVAL"),       # unknown scope
                       ((data, flags, 256, 1, 4, 1, 1), "EUNSUPPORTED")):  # 512 WGs > CUs
        with pytest.raises(pkg.SymtileError) as e:
            pkg.symtile_litmus_mp(heap.handle, *args, 0, res.data_ptr(), pkg.current_stream())
        assert e.value.name == name, args
    for args, name in (((flags, 0, 1, 1, 1), "EINVAL"),                  # no pairs
                       ((flags + 4, 1, 1, 1, 1), "EINVAL"),              # misaligned
                       ((flags, 1, 1, 3, 1), "EINVAL"),                  # unknown form
                       ((flags, 256, 1, 1, 1), "EUNSUPPORTED")):
        with pytest.raises(pkg.SymtileError) as e:
            pkg.symtile_litmus_sb(heap.handle, *args, 0, res.data_ptr(), pkg.current_stream())
        assert e.value.name == name, args
    heap.barrier()


@pytest.mark.parametrize("mode", [0, 1], ids=["put", "get"])
@pytest.mark.parametrize("case", [
    # world, rows, cols, tile_r, tile_c, dtype: odd counts of tiles a row, runs of
    # unequal length, widths that are no power of two, one tile row, wide tiles
    (4, 300, 1160, 64, 64, "bf16"), (2, 130, 2040, 64, 24, "f16"), (8, 33, 260, 32, 4, "f32"),
    (3, 64, 8, 64, 8, "bf16"), (1, 70, 1000, 7, 40, "f32"), (2, 20, 16384, 16, 16384, "f32"),
    (2, 9, 12304, 8, 4104, "bf16"), (8, 520, 2048, 128, 128, "f32"),
    # tiles that leave waves of a workgroup without a chunk, tiles wider than the matrix
    (2, 200, 24, 8, 8, "bf16"), (4, 100, 48, 15, 24, "bf16"), (2, 64, 64, 64, 1 << 28, "f32"),
], ids=lambda c: "w%d_%dx%d_t%dx%d_%s" % c)
def test_heap_tile_copy_automatic_runs(case, mode):
    """The library's own split of the tile rows into runs, and the caller's (one,
    three and all tiles of a row per workgroup), for all ranks and one, with shifts
    of either sign: every byte and counter as the oracle's copy leaves them."""
    pkg = sym()
    world, rows, cols, tr, tc, dt = case
    tdt = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}[dt]
    code = {"bf16": pkg.BF16, "f16": pkg.F16, "f32": pkg.F32}[dt]
    ival = torch.int16 if dt != "f32" else torch.int32
    heap, src, dst, flags = _copy_heap(pkg, world, rows, cols, tdt)
    g = torch.Generator().manual_seed(5)
    send = torch.randint(-2 ** 15, 2 ** 15, (world, rows, cols), generator=g).to(ival)
    heap.slots_view(src, (rows, cols), ival).copy_(send.cuda())
    tiles_c = -(-cols // tc)
    ntiles = -(-rows // tr) * tiles_c
    for only, shift, per in ((-1, 1, 0), (world - 1, -1, 0), (-1, -world - 2, 1), (-1, 2, 3),
                             (0, 1, tiles_c)):
        heap.slots_view(flags, (ntiles,), torch.int32).zero_()
        heap.slots_view(dst, (rows, cols), ival).zero_()
        pkg.symtile_tile_copy(heap.handle, src, dst, rows, cols, cols, code, tr, tc, shift, only,
                              flags, tiles_per_wg=per, stream=pkg.current_stream(), mode=mode)
        heap.barrier()
        recv = heap.slots_view(dst, (rows, cols), ival).cpu().numpy()
        fl = heap.slots_view(flags, (ntiles,), torch.int32).cpu().numpy()
        want, wf = oracle.tile_copy(send.numpy(), np.zeros_like(send.numpy()), tr, tc, shift,
                                    only_rank=only, get=bool(mode))
        assert np.array_equal(recv, want), (only, shift, per)
        assert np.array_equal(fl, wf.astype(np.int32)), (only, shift, per)


def test_heap_tile_copy_two_gib_call():
    """From 2 GiB read and written on the tile rows are cut into narrow runs: every
    block and counter as for smaller calls (rows and columns end inside a tile)."""
    pkg = sym()
    world, rows, cols, t = 8, 4100, 8200, 128
    heap, src, dst, flags = _copy_heap(pkg, world, rows, cols, torch.float32)
    send = heap.slots_view(src, (rows, cols), torch.int32)
    for r in range(world):
        send[r].random_(-2 ** 31, 2 ** 31)
    tiles = (-(-rows // t), -(-cols // t))
    heap.slots_view(dst, (rows, cols), torch.int32).zero_()
    heap.slots_view(flags, tiles, torch.int32).zero_()
    pkg.symtile_tile_copy(heap.handle, src, dst, rows, cols, cols, pkg.F32, t, t, 3, -1, flags,
                          stream=pkg.current_stream())
    heap.barrier()
    recv = heap.slots_view(dst, (rows, cols), torch.int32)
    for r in range(world):
        assert torch.equal(recv[(r + 3) % world], send[r]), r
    assert bool((heap.slots_view(flags, tiles, torch.int32) == 1).all())
