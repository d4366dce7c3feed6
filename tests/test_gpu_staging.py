"""Both staging-copy paths against the oracle (GPU).

By default a library kernel stages each run of chunks from pinned host memory
into the ring; BSR_FLAG_SDMA_COPIES selects the copy engine instead, and a
store arena that HIP does not report pinned is always copied by the copy
engine.  Each path must leave the same bytes as the oracle.
"""

import numpy as np
import pytest
import torch

import oracle
from gpu_side import ROUTES, GpuCase, check_route, layout_of, say
from oracle_side import build_case
from paper_2608_17826_amd import bsr
from paper_2608_17826_amd.session import RestoreSession, group_dsts
from workloads import generate, get_config
from workloads.configs import GroupSpec, Workload
from workloads.device import place
from workloads.gen import random_workload

pytestmark = pytest.mark.gpu


def _oracle(wi, W):
    case = build_case(wi)
    n, _, keys = oracle.probe(case.store, wi.tokens, wi.workload.chunk_tokens, wi.salt)
    res = oracle.windowed_restore(case.layout, case.store, keys, n, W, wi.block_tables, case.pools, case.valid)
    return case, n, res


def _check(wi, case, res, out, pools, valid):
    assert out.exposed_tokens == res.exposed_tokens and out.fallback == 0
    assert out.stats["h2d_bytes"] == res.h2d_bytes
    for g in range(len(wi.workload.groups)):
        np.testing.assert_array_equal(valid[g].cpu().numpy(), case.valid[g])
        got = np.stack([p.cpu().numpy() for p in pools[g]])
        np.testing.assert_array_equal(got, case.pools[g], err_msg=f"pool of group {g}")


@pytest.mark.parametrize("W,batch", [(32, 0), (8, 0), (8, 8)])
def test_copy_engine_staging_parity(W, batch):
    wi = generate(get_config(2))
    say(f"case: workload 2 (32K), W={W}, batch={batch}, copy-engine staging")
    case, n, res = _oracle(wi, W)
    gc = GpuCase(wi, W=W, install_batch=batch, flags=bsr.BSR_FLAG_SDMA_COPIES)
    try:
        assert gc.probe(1)[0] == n
        out = gc.restore(1, n)
        _check(wi, case, res, out, gc.dev.pools, gc.dev.valid)
        assert out.stats["n_stage_launches"] == 0
    finally:
        gc.close()


@pytest.mark.parametrize("seed", [1, 4, 9, 13])
def test_copy_engine_staging_random_layouts(seed):
    w = random_workload(seed)
    wi = generate(w)
    W = w.windows[0]
    say(f"case: random layout seed={seed}, W={W}, copy-engine staging")
    case, n, res = _oracle(wi, W)
    gc = GpuCase(wi, W=W, flags=bsr.BSR_FLAG_SDMA_COPIES)
    try:
        out = gc.restore(2, gc.probe(2)[0])
        _check(wi, case, res, out, gc.dev.pools, gc.dev.valid)
    finally:
        gc.close()


@pytest.mark.parametrize("arena", ["pageable", "pinned"])
def test_adopted_arena(arena):
    """A caller arena: pageable memory (numpy) is copied by the copy engine;
    pinned memory (torch's pinned allocator) by the staging kernel.  Either
    way the image is the oracle's."""
    wi = generate(get_config(2))
    w = wi.workload
    say(f"case: workload 2 (32K), W=32, adopted {arena} arena")
    case, n, res = _oracle(wi, 32)
    layout = layout_of(wi)
    ctx = bsr.bsr_ctx_create(layout, 32, hip_device=0)
    try:
        stride = (bsr.bsr_slot_bytes(layout) + 4095) // 4096 * 4096
        nbytes = stride * (w.held_chunks + 1)
        if arena == "pageable":
            buf = np.zeros(nbytes, dtype=np.uint8)
            addr = buf.ctypes.data
        else:
            buf = torch.empty(nbytes, dtype=torch.uint8, pin_memory=True)
            addr = buf.data_ptr()
        bsr.bsr_store_adopt(ctx, addr, nbytes)
        keys = bsr.bsr_chunk_keys(wi.salt, wi.tokens, w.chunk_tokens)
        bsr.bsr_store_put_chunks(ctx, [int(k) for k in keys[:w.held_chunks]],
                                 [wi.payloads(i) for i in range(w.held_chunks)])
        dev = place(wi)
        torch.cuda.synchronize()
        sess = RestoreSession(ctx)
        got_n = bsr.bsr_probe(ctx, 3, wi.salt, wi.tokens)[0]
        assert got_n == n
        out = sess.restore(3, n, group_dsts(dev.block_tables, dev.tensor_bases, dev.valid, wi.pool_blocks))
        _check(wi, case, res, out, dev.pools, dev.valid)
        if arena == "pageable":
            assert out.stats["n_stage_launches"] == 0
        else:
            assert out.stats["n_stage_launches"] > 0 and out.stats["stage_bytes"] == res.h2d_bytes
        bsr.bsr_request_end(ctx, 3)
    finally:
        bsr.bsr_ctx_destroy(ctx)


def test_staging_kernel_link_rate_reported():
    """The staging kernel's own link measurement runs and reports a rate in
    the range of the copy engine's (both read the same pinned memory)."""
    wi = generate(get_config(1))
    ctx = bsr.bsr_ctx_create(layout_of(wi), 2, hip_device=0)
    try:
        k = bsr.bsr_measure_stage(ctx, 256 << 20, 3)
        e = bsr.bsr_measure_h2d(ctx, 256 << 20, 1, 3)
        say(f"staging kernel {k:.1f} GB/s, copy engine {e:.1f} GB/s")
        assert k > 0.5 * e and e > 0
        with pytest.raises(bsr.BsrError):
            bsr.bsr_measure_stage(ctx, 1000, 1)      # not a multiple of 16
    finally:
        bsr.bsr_ctx_destroy(ctx)


def test_scatter_ceiling_measurement():
    """The plain scattered-copy ceiling runs for the layouts' block sizes,
    cold and warm, and rejects block sizes that are not 16-byte multiples."""
    wi = generate(get_config(1))
    ctx = bsr.bsr_ctx_create(layout_of(wi), 2, hip_device=0)
    try:
        for bb in (73_728, 16_896, 16_384):
            cold = bsr.bsr_measure_scatter(ctx, bb, 64 << 20, 2, 1)
            warm = bsr.bsr_measure_scatter(ctx, bb, 64 << 20, 2, 1, bsr.BSR_SCATTER_WARM_SOURCE)
            say(f"{bb} B blocks: {cold:.0f} GB/s cold, {warm:.0f} GB/s warm")
            assert cold > 100 and warm > 100
        with pytest.raises(bsr.BsrError):
            bsr.bsr_measure_scatter(ctx, 1000, 64 << 20, 1, 1)
        with pytest.raises(bsr.BsrError):
            bsr.bsr_measure_scatter(ctx, 16_384, 64 << 20, 1, 1, 2)     # unknown flag
    finally:
        bsr.bsr_ctx_destroy(ctx)


def test_timing_flags_are_taken_at_bind():
    """BSR_FLAG_TIME_INSTALL stamps installs only, BSR_FLAG_TIME_STAGE the
    staging launches only; bsr_set_timing changes them for requests bound
    afterwards, never for one already bound."""
    wi = generate(get_config(2))
    say("case: workload 2 (32K), W=32, timing flags per request")
    case, n, res = _oracle(wi, 32)
    gc = GpuCase(wi, W=32, flags=bsr.BSR_FLAG_TIME_INSTALL)
    try:
        def restore(rid, **kw):
            assert gc.probe(rid)[0] == n
            out = gc.restore(rid, n, **kw)
            _check(wi, case, res, out, gc.dev.pools, gc.dev.valid)
            bsr.bsr_request_end(gc.ctx, rid)
            return out.stats

        st = restore(31)
        assert st["install_ms_total"] > 0 and st["n_stage_launches"] > 0 and st["stage_ms_total"] == 0
        bsr.bsr_set_timing(gc.ctx, bsr.BSR_FLAG_TIME_STAGE)
        st = restore(32)
        assert st["install_ms_total"] == 0 and st["stage_ms_total"] > 0
        # changed while bound: this request keeps the flags of its bind
        st = restore(33, after_bind=lambda: bsr.bsr_set_timing(gc.ctx, bsr.BSR_FLAG_TIME_INSTALL))
        assert st["install_ms_total"] == 0 and st["stage_ms_total"] > 0
        st = restore(34)
        assert st["install_ms_total"] > 0 and st["stage_ms_total"] == 0
        with pytest.raises(bsr.BsrError):
            bsr.bsr_set_timing(gc.ctx, bsr.BSR_FLAG_SDMA_COPIES)
    finally:
        gc.close()


# (record bytes, chunk tokens): slots of 256 B, one tile (4,096 B), a tile and
# one 256 B part, and three tiles and a part, none adjacent in the arena but
# the second
@pytest.mark.parametrize("flags", ROUTES)
@pytest.mark.parametrize("record,C,W", [(4, 8, 3), (128, 32, 8), (124, 35, 40), (1152, 11, 33)])
def test_runs_of_a_scattered_store(record, C, W, flags):
    """Chunks stored one by one in a random order.  Through the ring, a staging
    launch takes many runs (up to 32, in one window of more) of one to a few
    chunks each, so there are fewer launches than chunks: one per batch, one
    for the rest of a window, and one more where the slots of a batch are
    released by two earlier ones.  Straight from pinned memory, a launch reads
    chunks from all over the arena.  The image is the oracle's either way."""
    w = Workload(index=400 + record, name="runs", n_tokens=70 * C + 3, chunk_tokens=C,
                 groups=(GroupSpec("g", 8, 1, record, value_kind="bytes"),), windows=(W,), pool_factor=2)
    wi = generate(w)
    case, n, res = _oracle(wi, W)
    say(f"case: 70 chunks of {bsr.bsr_slot_bytes(layout_of(wi))} B stored in random order, W={W}, flags={flags}")
    gc = GpuCase(wi, W=W, flags=flags, pinned_chunks=[], arena_chunks=72)
    try:
        for i in np.random.default_rng(record).permutation(70):
            bsr.bsr_store_put_chunk(gc.ctx, int(gc.keys[i]), wi.payloads(int(i)))
        assert gc.probe(5)[0] == n == 70
        out = gc.restore(5, n)
        _check(wi, case, res, out, gc.dev.pools, gc.dev.valid)
        check_route(gc.ctx, 5, out.stats, flags)
        batches = -(-70 // out.stats["install_batch"])
        assert out.stats["n_stage_launches"] <= min(69, 2 * batches + out.stats["n_windows"])
    finally:
        gc.close()


def _direct_workload(groups, C, n_chunks, W):
    specs = tuple(GroupSpec(f"g{i}", bt, nt, rb, kind="planar" if sp else "contig", split_bytes=sp,
                            value_kind="bytes") for i, (bt, nt, rb, sp) in enumerate(groups))
    return Workload(index=500, name="direct", n_tokens=n_chunks * C + 1, chunk_tokens=C, groups=specs,
                    windows=(W,), pool_factor=2)


# one piece; a piece and one vector more; more pieces than workgroups; records
# and blocks that leave nothing 16-byte aligned, in pieces of up to 8 KiB and
# planar ones of more than the 8 KiB in flight; planar pieces through the LDS
# one after the other in a workgroup
DIRECT = [([(16, 1, 16, 0)], 16, 1, 1), ([(64, 1, 132, 0)], 64, 33, 2), ([(64, 9, 1152, 0)], 64, 40, 32),
          ([(5, 4, 1148, 0), (7, 8, 140, 132)], 48, 34, 3), ([(128, 2, 132, 124), (64, 1, 2044, 0)], 128, 5, 0),
          ([(128, 40, 132, 128), (16, 1, 48, 0)], 256, 9, 8)]


@pytest.mark.parametrize("groups,C,n_chunks,W", DIRECT)
@pytest.mark.parametrize("bad", [None, "first", "last"])
def test_install_straight_from_pinned_memory(groups, C, n_chunks, W, bad):
    """A small request's chunks go from the pinned store to their blocks with
    no staging copy; a corrupt word in the first or last chunk is found by the
    launch that holds it, as in the oracle."""
    w = _direct_workload(groups, C, n_chunks, W)
    wi = generate(w)
    k, g = (0 if bad == "first" else n_chunks - 1), len(groups) - 1
    case = build_case(wi)
    n, _, keys = oracle.probe(case.store, wi.tokens, C, wi.salt)
    byte = case.layout.payload_bytes(g) - 3
    if bad:
        case.store.corrupt(keys[k], g, byte, 0x81)
    res = oracle.windowed_restore(case.layout, case.store, keys, n, W, wi.block_tables, case.pools, case.valid)
    say(f"case: direct install, {groups}, C={C}, {n_chunks} chunks, W={W}, corrupt {bad}")
    gc = GpuCase(wi, W=W)
    try:
        assert gc.probe(6)[0] == n == n_chunks
        if bad:
            gc.corrupt(int(keys[k]), g, byte, 0x81)
        out = gc.restore(6, n)
        assert out.stats["n_stage_launches"] == 0
        assert out.status["fail"] == (bsr.BSR_FAIL_CORRUPT if bad else 0) and out.fallback == res.fallback
        assert out.status["first_failed_chunk"] == res.first_failed_chunk
        assert out.status["q"][:len(groups)] == res.q
        if not bad:
            _check(wi, case, res, out, gc.dev.pools, gc.dev.valid)
            return
        bsr.bsr_request_end(gc.ctx, 6)
        gc.corrupt(int(keys[k]), g, byte, 0x81)  # put back: the shared words were left as a launch needs them
        assert gc.probe(7)[0] == n and gc.restore(7, n).exposed_tokens == n * C
    finally:
        gc.close()


# records larger than the registers hold, beside unaligned ones; a planar piece
# that fits them only when it starts on a vector (tensor 0 does, 1 does not);
# planes whose values are no whole vectors; eight groups in enough pieces for
# workgroups to take stretches of them, in launches of 32 and of 13 chunks
DIRECT_PIECES = [([(4, 1, 24_000, 128), (3, 2, 20, 0)], 4, 9, 4), ([(2048, 2, 20, 16)], 1027, 3, 2),
                 ([(16, 2, 28, 12), (48, 1, 2048, 0)], 24, 7, 3),
                 ([(8, 2, 64, 0), (16, 1, 36, 32), (64, 3, 20, 0), (24, 2, 132, 128), (32, 1, 1152, 0), (5, 2, 12, 0),
                   (48, 1, 24, 8), (128, 2, 512, 0)], 32, 45, 32)]


@pytest.mark.parametrize("groups,C,n_chunks,W", DIRECT_PIECES)
@pytest.mark.parametrize("bad", [None, "last"])
def test_direct_pieces_at_the_limits_of_the_registers(groups, C, n_chunks, W, bad):
    test_install_straight_from_pinned_memory(groups, C, n_chunks, W, bad)


def test_direct_and_staged_chunks_in_one_request(tmp_path):
    """Runs of chunks from the pinned store and from files alternate: the
    former are installed straight from there, the latter through the ring."""
    w = _direct_workload([(16, 3, 132, 0), (32, 2, 132, 128)], 32, 40, 6)
    wi = generate(w)
    case, n, res = _oracle(wi, 6)
    pinned = [i for i in range(40) if (i // 3) % 2 or i > 33]
    say("case: 40 chunks, three pinned, three in files, and so on, W=6")
    gc = GpuCase(wi, W=6, pinned_chunks=pinned, flags=bsr.BSR_FLAG_TIME_INSTALL)
    try:
        gc.put_files(str(tmp_path), [i for i in range(40) if i not in pinned])
        assert gc.probe(8)[0] == n == 40
        out = gc.restore(8, n)
        _check(wi, case, res, out, gc.dev.pools, gc.dev.valid)
        assert out.stats["file_tier_chunks"] == 40 - len(pinned) == out.stats["n_stage_launches"]
        assert out.stats["install_batch"] == 6      # of the ring's launches
        d = bsr.bsr_direct_stats(gc.ctx, 8)
        assert 0 < d["n_launches"] < out.stats["n_install_launches"] and 0 < d["ms_total"] < out.stats["install_ms_total"]
        assert d["bytes"] * 40 == len(pinned) * out.stats["installed_bytes"]
        assert gc.probe(9)[0] == n
        with pytest.raises(bsr.BsrError) as e:
            bsr.bsr_direct_stats(gc.ctx, 9)         # probed only
        assert e.value.code == bsr.BSR_E_NOTFOUND
    finally:
        gc.close()


@pytest.mark.parametrize("n_chunks,in_file,staged", [(64, 0, 0), (65, 0, 0), (65, 1, 65), (65, 64, 65)])
def test_requests_beyond_64_mib(tmp_path, n_chunks, in_file, staged):
    """Chunks of 1 MiB.  A request of more than 64 of them is installed
    straight from pinned memory if all are there; with any in a file its
    chunks go through the ring, on two streams."""
    w = _direct_workload([(64, 4, 1024, 0)], 256, n_chunks, 8)
    wi = generate(w)
    case, n, res = _oracle(wi, 8)
    say(f"case: {n_chunks} chunks of 1 MiB, the last {in_file} in files, W=8")
    first_file = n_chunks - in_file
    gc = GpuCase(wi, W=8, pinned_chunks=range(first_file))
    try:
        if in_file:
            gc.put_files(str(tmp_path), range(first_file, n_chunks))
        assert gc.probe(8)[0] == n == n_chunks
        out = gc.restore(8, n)
        _check(wi, case, res, out, gc.dev.pools, gc.dev.valid)
        assert out.stats["file_tier_chunks"] == in_file and out.stats["stage_bytes"] == staged << 20
    finally:
        gc.close()


@pytest.mark.parametrize("n_chunks", [12, 70])
@pytest.mark.parametrize("fault", ["corrupt", "marked", "aborted", "launch"])
def test_direct_requests_fail_closed(n_chunks, fault):
    """Chunks of 1 MiB, installed straight from pinned memory: 12 on the
    compute stream, 70 by launches on the copy stream.  A corrupt entry in the
    last chunk, a group marked invalid or the request aborted after its second
    window, or a failed launch (forced from the host; the chunks it kept are
    installed before the commit's invalidation): the outcome is the oracle's,
    and the same context restores the request afterwards."""
    W = 4 if n_chunks < 64 else 16
    w = _direct_workload([(64, 3, 1024, 0), (64, 1, 1024, 0)], 256, n_chunks, W)
    wi = generate(w)
    case = build_case(wi)
    n, _, keys = oracle.probe(case.store, wi.tokens, 256, wi.salt)
    kw = {}
    if fault == "corrupt":
        case.store.corrupt(keys[n - 1], 1, 4097, 0x42)
    elif fault == "marked":
        kw["invalid_groups"] = [1]
    elif fault == "aborted":
        kw["abort_after_windows"] = 2
    else:
        kw["faults"] = {W: oracle.FAIL_TRANSFER}
    res = oracle.windowed_restore(case.layout, case.store, keys, n, W, wi.block_tables, case.pools, case.valid, **kw)
    say(f"case: direct installs of {n_chunks} chunks of 1 MiB, W={W}, {fault}")
    gc = GpuCase(wi, W=W)
    try:
        assert gc.probe(8)[0] == n == n_chunks
        if fault == "corrupt":
            gc.corrupt(int(keys[n - 1]), 1, 4097, 0x42)
        if fault == "launch":
            bsr.bsr_debug_inject(gc.ctx, bsr.BSR_INJECT_LAUNCH_ERROR, W, 0)

        def mark(j):
            if fault == "marked" and j == 1:
                bsr.bsr_mark_group_invalid(gc.ctx, 8, 1)
        out = gc.restore(8, n, after_window=mark, abort_after_windows=kw.get("abort_after_windows"))
        assert out.exposed_tokens == res.exposed_tokens == 0 and out.fallback == 1
        if fault == "launch":
            assert [c for _, c in out.window_errors] == [bsr.BSR_E_TRANSFER]
            assert out.status["fail"] == bsr.BSR_FAIL_TRANSFER
        else:
            assert out.status["first_failed_chunk"] == res.first_failed_chunk and out.status["q"][:2] == res.q
        for g in range(2):
            np.testing.assert_array_equal(gc.valid_host(g), case.valid[g])
        check_route(gc.ctx, 8, out.stats, 0)
        assert gc.probe(8)[0] == 0          # force-local after the fallback
        bsr.bsr_request_end(gc.ctx, 8)
        if fault == "corrupt":
            gc.corrupt(int(keys[n - 1]), 1, 4097, 0x42)
        case, n, res = _oracle(wi, W)
        assert gc.probe(9)[0] == n
        _check(wi, case, res, gc.restore(9, n), gc.dev.pools, gc.dev.valid)
    finally:
        gc.close()


@pytest.mark.parametrize("n_chunks", [1, 64, 1024, 1025])
def test_bind_checks_the_last_block_id(n_chunks):
    """Block tables of 16 to 16,400 entries over two groups, read back in one
    launch up to 16,384 and by copies beyond: an id past the pool or a
    repeated one in the very last entry is refused, with the valid bytes as
    they were, and the same tables put right restore the oracle's image."""
    w = Workload(index=600, name="tables", n_tokens=n_chunks * 16, chunk_tokens=16,
                 groups=(GroupSpec("a", 16, 1, 8, value_kind="bytes"), GroupSpec("b", 1, 1, 4, value_kind="bytes"))
                 if n_chunks < 1024 else (GroupSpec("b", 1, 1, 4, value_kind="bytes"),),
                 windows=(32,), pool_factor=2)
    wi = generate(w)
    case, n, res = _oracle(wi, 32)
    gc = GpuCase(wi, W=32)
    try:
        say(f"case: {sum(len(t) for t in wi.block_tables)} block table entries")
        assert gc.probe(9)[0] == n == n_chunks
        table, good = gc.dev.block_tables[-1], int(wi.block_tables[-1][-1])
        for bad, word in ((wi.pool_blocks[-1], "outside"), (-1, "outside"), (int(wi.block_tables[-1][0]), "twice")):
            table[-1] = bad
            torch.cuda.synchronize()
            with pytest.raises(bsr.BsrError) as e:
                gc.session.bind(9, n, gc.dsts())
            assert e.value.code == bsr.BSR_E_ARG and word in str(e.value)
            np.testing.assert_array_equal(gc.valid_host(len(w.groups) - 1), wi.valid_init[-1])
        table[-1] = good
        torch.cuda.synchronize()
        with torch.cuda.stream(gc.session.compute_stream):
            torch.cuda._sleep(2_000_000)  # the readback then waits for the stream, past its polling
        _check(wi, case, res, gc.restore(9, n), gc.dev.pools, gc.dev.valid)
    finally:
        gc.close()


@pytest.mark.parametrize("batch", [0, 8])
@pytest.mark.parametrize("paused", [True, False])
def test_direct_chunks_wait_only_while_the_device_is_busy(batch, paused):
    """Windows of two 1 MiB chunks.  A caller that lets the device finish
    between windows has every window launched by its own call, whatever
    install_batch allows; while the device is busy (a spin kernel ahead on the
    compute stream) launches double: the third window waits for the fourth,
    the fifth for the last."""
    w = _direct_workload([(64, 4, 1024, 0)], 256, 12, 8)
    wi = generate(w)
    case, n, res = _oracle(wi, 8)
    say(f"case: 12 chunks of 1 MiB in windows of 2, install_batch {batch}, {'paused' if paused else 'busy'}")
    gc = GpuCase(wi, W=8, install_batch=batch)
    launches = []
    try:
        assert gc.probe(8)[0] == n == 12

        def busy():
            if not paused:
                with torch.cuda.stream(gc.session.compute_stream):
                    torch.cuda._sleep(100_000_000)  # far longer than the calls take

        def after(j):
            launches.append(bsr.bsr_request_stats(gc.ctx, 8)["n_install_launches"])
            if paused:
                gc.session.compute_stream.synchronize()
                gc.session.copy_stream.synchronize()
        out = gc.restore(8, n, plan=[(i, 2) for i in range(0, 12, 2)], after_bind=busy, after_window=after)
        _check(wi, case, res, out, gc.dev.pools, gc.dev.valid)
        assert launches == ([1, 2, 3, 4, 5, 6] if paused else [1, 2, 2, 3, 3, 4])
    finally:
        gc.close()


@pytest.mark.parametrize("n_chunks", [12, 70])
def test_direct_installs_under_capture(n_chunks):
    """The windows of a bound request captured into a graph from the compute
    stream (chunks of 1 MiB: 12 on that stream alone, 70 with launches on the
    copy stream, joined again when the prefix is complete).  Nothing is
    installed until the graph is launched; then the commit exposes the
    oracle's image."""
    w = _direct_workload([(64, 4, 1024, 0)], 256, n_chunks, 16)
    wi = generate(w)
    case, n, res = _oracle(wi, 16)
    say(f"case: {n_chunks} chunks of 1 MiB, W=16, windows captured")
    gc = GpuCase(wi, W=16)
    try:
        assert gc.probe(8)[0] == n == n_chunks
        sess, graph = gc.session, torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        sess.bind(8, n, gc.dsts())
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=sess.compute_stream, capture_error_mode="thread_local"):
            for first, cnt in sess.next_windows(8):
                bsr.bsr_restore_window(gc.ctx, 8, first, cnt)
        np.testing.assert_array_equal(gc.pool_host(0), wi.sentinel_pool(0))
        with torch.cuda.stream(sess.compute_stream):
            graph.replay()
        _check(wi, case, res, sess.commit(8), gc.dev.pools, gc.dev.valid)
    finally:
        gc.close()
