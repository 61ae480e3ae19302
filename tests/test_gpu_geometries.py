"""GPU parity on geometries at the edges of what the format allows: 1- and
4-byte elements, an odd number of rows per chunk, the maximum layer count
(metadata larger than one LDS tile), a 4 MiB slab (64 chunks per slab), and a
single block. Save and restore are compared with the oracle byte for byte,
with damaged records in the restore."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import taliesin_ref as ref
from paper_2609_39358_amd.device import PagedCache
from tests.gpu_case import DEV, Case, host_layers, i64, log, random_fill
from tests.test_gpu_parity import check_restore, upload_records

pytestmark = pytest.mark.gpu

GEOMS = {
    "fp8": (wl.Geometry(3, 8, 128, 16, "fp8"), 6),
    "f32": (wl.Geometry(2, 2, 32, 16, "f32"), 6),
    "odd_rows_p13": (wl.Geometry(2, 8, 64, 13), 6),
    "max_layers": (wl.Geometry(256, 1, 32, 16), 3),
    "slab_4MiB": (wl.Geometry(1, 16, 256, 512), 3),
    "one_block": (wl.Geometry(4, 4, 64, 16), 1),
}


@pytest.mark.parametrize("name", list(GEOMS))
def test_edge_geometry_round_trip(name):
    geom, n = GEOMS[name]
    c = Case(geom, n, n + 2, n + 3, seed=17)
    lay = c.lay
    log("geometry", name, "slab", lay.slab_bytes, "chunks/slab", lay.chunks_per_slab, "meta", lay.meta_bytes)
    c.make_src()
    store, st = c.save()
    recs_o, st_o = c.oracle_save()
    assert [int(x) for x in st] == st_o
    got = store.buf.cpu().numpy()
    for b in range(n):
        assert got[b].tobytes() == recs_o[b], b
    recs = [bytearray(r) for r in recs_o]
    rb, po = lay.record_bytes, lay.payload_offset
    if n > 1:
        recs[1][po + (rb - po) // 3] ^= 0x01  # a payload chunk in the middle
    if n > 2:
        recs[2][lay.meta_bytes - 300] ^= 0x80  # late in the metadata (token ids / padding)
    store2 = upload_records(recs, rb)
    dst = random_fill(PagedCache(geom.n_layers, n + 3, c.stride, DEV), 3)
    hk0, hv0 = host_layers(dst)
    vo = check_restore(c, [bytes(r) for r in recs], store2.ptrs, store2.lens, c.t_dst, dst, hk0, hv0)
    assert vo[0] == ref.ACCEPT
    if n > 1:
        assert vo[1] == ref.SEGMENT
    if n > 2:
        assert vo[2] == ref.ROOT


@pytest.mark.parametrize("name", list(GEOMS))
def test_edge_geometry_shared_save(name):
    """The save kernel for running beside other work (TL_SAVE_SHARED) writes
    the oracle's records on every edge geometry, in one layer range and in
    one-layer parts."""
    from paper_2609_39358_amd import taliesin as T
    from paper_2609_39358_amd.device import RecordStore
    from tests.gpu_case import i32
    geom, n = GEOMS[name]
    c = Case(geom, n, n + 2, n + 3, seed=19)
    c.make_src()
    recs_o, st_o = c.oracle_save()
    blk = c.blocks(i32(c.t_src))
    s = torch.cuda.current_stream()
    L = geom.n_layers
    for parts in ([(0, L)], [(l, l + 1) for l in range(L)][::-1]):
        store = RecordStore(n, c.lay.record_bytes, DEV)
        store.buf.fill_(0xA5)
        for a, b in parts:
            T.tl_save_layers(c.ctx, s, n, c.src.tl(), blk, store.ptrs, a, b, shared=True)
        st = torch.zeros(n, dtype=torch.uint8, device=DEV)
        T.tl_save_seal(c.ctx, s, n, c.src_pages, blk, store.ptrs, st)
        torch.cuda.synchronize()
        assert [int(x) for x in st.cpu()] == st_o
        got = store.buf.cpu().numpy()
        for b in range(n):
            assert got[b].tobytes() == recs_o[b], (len(parts), b)


# Blocks of 1 KiB slabs with digest tables on both sides of the length from
# which a save hashes them beside the copy: 8,188 (one launch), 8,192 and 10,000
# digests; the last case also ends in a partial block and holds a refused block
# and a missing record, whose digests are never made.
@pytest.mark.parametrize("layers,ppb,n,odd", [(2, 2047, 1, False), (2, 2048, 1, False), (2, 2048, 3, False),
                                              (1, 5000, 4, True)])
def test_long_digest_tables(layers, ppb, n, odd):
    from paper_2609_39358_amd import taliesin as T
    from paper_2609_39358_amd.device import RecordStore
    from tests.gpu_case import i32
    geom = wl.Geometry(layers, 1, 64, 8, pages_per_block=ppb)
    c = Case(geom, n, n * ppb + 5, n * ppb + 5, seed=23)
    c.make_src()
    counts = np.full(n, geom.block_tokens, np.int32)
    tables = c.t_src.copy()
    ptr_on = np.ones(n, bool)
    if odd:
        counts[3] = 8 * 3001 + 3  # pages 3,002.. of the last block hold no tokens
        tables[:, 3 * ppb + 3002:] = -1
        tables[:, 1 * ppb + 4321] = c.src_pages
        ptr_on[2] = False
        c.tokens[3, counts[3]:] = 0
        c.d_tokens = i32(c.tokens.view(np.int32))
    hk, hv = host_layers(c.src)
    recs_o, st_o = ref.save(c.lay, c.ns, hk, hv, tables, [k.tobytes() for k in c.keys], c.bidx, c.tokens,
                            n_pages=c.src_pages, n_tokens=counts)
    store = RecordStore(n, c.lay.record_bytes, DEV)
    store.buf.fill_(0xA5)
    ptrs = store.ptrs * torch.from_numpy(ptr_on.astype(np.int64)).to(DEV)
    st = torch.zeros(n, dtype=torch.uint8, device=DEV)
    blk = T.make_blocks(c.d_keys, c.d_bidx, c.d_tokens, i32(tables), i32(counts))
    log("long digest tables", layers, "x", ppb, "pages,", n, "blocks")
    for _ in range(2):  # the second save overwrites whole records
        T.tl_save(c.ctx, torch.cuda.current_stream(), n, c.src.tl(), blk, ptrs, st)
    torch.cuda.synchronize()
    got, st = store.buf.cpu().numpy(), [int(x) for x in st.cpu()]
    for b in range(n):
        if ptr_on[b]:
            assert st[b] == st_o[b] and got[b].tobytes() == recs_o[b], b
        else:
            assert st[b] == T.MISSING and (got[b] == 0xA5).all(), b


# A call may name one record several times, for the same block (requests of one
# batch that share it): all of them write the same bytes. Records with long
# digest tables are hashed while others of the call are copied: blocks of one
# record that are whole by then, not begun, and in between.
@pytest.mark.parametrize("ppb,same", [(2048, [0, 0]), (2048, [0, 1, 0, 1, 2]), (5000, [0, 0, 0]), (7001, [0, 1, 1, 0]),
                                      (64, [0, 0, 1])])
def test_blocks_of_one_record(ppb, same):
    from paper_2609_39358_amd import taliesin as T
    from paper_2609_39358_amd.device import RecordStore
    from tests.gpu_case import i32
    geom = wl.Geometry(2, 1, 64, 8, pages_per_block=ppb)
    n = len(same)
    c = Case(geom, n, n * ppb, n * ppb, seed=41, block_index=same)
    c.make_src()
    c.tokens = np.ascontiguousarray(c.tokens[same])
    c.keys = np.ascontiguousarray(c.keys[same])
    tables = np.concatenate([c.t_src[:, b * ppb:(b + 1) * ppb] for b in same], axis=1)
    recs_o, st_o = ref.save(c.lay, c.ns, *host_layers(c.src), tables, [k.tobytes() for k in c.keys], c.bidx, c.tokens,
                            n_pages=c.src_pages)
    blk = T.make_blocks(torch.from_numpy(c.keys).to(DEV), c.d_bidx, i32(c.tokens.view(np.int32)), i32(tables))
    store = RecordStore(n, c.lay.record_bytes, DEV)
    ptrs = store.ptrs[torch.tensor(same, device=DEV)]
    st = torch.zeros(n, dtype=torch.uint8, device=DEV)
    log("blocks of one record", ppb, "pages,", same)
    for seed in range(3):  # the records' bytes before the save change nothing
        store.buf.random_(generator=torch.Generator(device=DEV).manual_seed(seed))
        T.tl_save(c.ctx, torch.cuda.current_stream(), n, c.src.tl(), blk, ptrs, st)
        torch.cuda.synchronize()
        assert [int(x) for x in st.cpu()] == st_o == [ref.ACCEPT] * n
        got = store.buf.cpu().numpy()
        for b, r in enumerate(same):
            assert got[r].tobytes() == recs_o[b], (b, r)


# Small blocks of at most 15 chunks are restored by one workgroup each (7 layers:
# 14 chunks), longer ones by the whole grid (8 layers: 16), whose pass over
# verdicts takes 1,024 blocks at a time: counts around that, with rejected
# blocks at its edges, and with every block rejected.
@pytest.mark.parametrize("layers,n,bad", [(7, 3, [0]), (8, 1, [0]), (8, 1023, [0, 1022]), (8, 1024, [1023]),
                                          (8, 1025, [1023, 1024]), (7, 1025, [0, 1024]),
                                          (8, 2100, [0, 255, 256, 1024, 2047, 2048, 2099]), (8, 1100, range(1100)),
                                          (8, 3500, [3, *range(1024, 2048), *range(2050, 2173), 3499])])
def test_rejected_blocks_at_tile_edges(layers, n, bad):
    geom = wl.Geometry(layers, 1, 64, 8)
    c = Case(geom, n, n, n + 3, seed=29)
    c.make_src()
    store, st = c.save()
    assert (st == ref.ACCEPT).all()
    recs = [bytearray(r.tobytes()) for r in store.buf.cpu().numpy()]
    for i, b in enumerate(bad):
        recs[b][(c.lay.payload_offset + 7) if i & 1 else 100] ^= 0x10
    store2 = upload_records(recs, c.lay.record_bytes)
    dst = random_fill(PagedCache(geom.n_layers, n + 3, c.stride, DEV), 3)
    hk0, hv0 = host_layers(dst)
    vo = check_restore(c, [bytes(r) for r in recs], store2.ptrs, store2.lens, c.t_dst, dst, hk0, hv0)
    assert sorted(b for b in range(n) if vo[b] != ref.ACCEPT) == sorted(bad)


# Requests whose ends are not stored: runs of missing blocks without pages among
# damaged ones with them, with up to 8 table entries per block and with more; a
# damaged block may have pages in one layer group or on its last page alone, and
# a missing one may have pages too.
@pytest.mark.parametrize("groups,ppb", [(1, 1), (2, 1), (2, 4), (1, 9), (3, 3)])
def test_rejected_blocks_among_missing_ones(groups, ppb):
    layers, n = 8, 1100 if ppb == 1 else 300
    geom = wl.Geometry(layers, 1, 64, 8, "bf16", (0,) * layers, tuple(l % groups for l in range(layers)), ppb)
    c = Case(geom, n, n * ppb, n * ppb + 3, seed=43)
    c.make_src()
    store, _ = c.save()
    recs = [bytearray(r.tobytes()) for r in store.buf.cpu().numpy()]
    t_dst, ptrs = c.t_dst.copy(), store.ptrs.clone()
    gone = [b for b in range(n) if b % 100 >= 60]
    for b in gone:
        recs[b] = None
        ptrs[b] = 0
        if b % 100 != 77:
            t_dst[:, b * ppb:(b + 1) * ppb] = -1
    for b in range(3, n, 50):
        if recs[b] is not None:
            recs[b][90] ^= 2
            if b % 100 < 50:  # one group's last page is all that is restored
                t_dst[:, b * ppb:(b + 1) * ppb - 1] = -1
                t_dst[:-1, (b + 1) * ppb - 1] = -1
    store2 = upload_records([r or b"" for r in recs], c.lay.record_bytes)
    ptrs += (store2.ptrs - store.ptrs) * (ptrs != 0)
    dst = random_fill(PagedCache(layers, n * ppb + 3, c.stride, DEV), 3)
    hk0, hv0 = host_layers(dst)
    log("rejected among missing", groups, "groups", ppb, "pages", n, "blocks")
    vo = check_restore(c, [None if r is None else bytes(r) for r in recs], ptrs, store2.lens, t_dst, dst, hk0, hv0)
    assert [b for b in range(n) if vo[b] == ref.MISSING] == gone and ref.ROOT in vo and ref.ACCEPT in vo


# Slabs of a 64-row chunk and a ragged one, in blocks of 4 chunks (a workgroup
# per block) and of 12 and 20, and of 1,024 of which 8 have 8,192 (whole chunks in
# flight), with pages that are not restored (nor read) and damage in a chunk of
# one that is.
@pytest.mark.parametrize("layers,n,rows", [(layers, 5, rows) for layers in (1, 3, 5) for rows in (65, 67, 96, 127)] +
                         [(256, 7, 65), (256, 8, 65), (256, 8, 79)])
def test_ragged_chunks_of_small_and_large_blocks(layers, n, rows):
    geom = wl.Geometry(layers, 2, 256, rows)
    c = Case(geom, n, n, n + 2, seed=31, stride_extra=48)
    c.make_src()
    store, _ = c.save()
    recs = [bytearray(r.tobytes()) for r in store.buf.cpu().numpy()]
    recs[1][c.lay.payload_offset + 70 * 1024 * layers] ^= 1
    recs[3][-3] ^= 0x40
    store2 = upload_records(recs, c.lay.record_bytes)
    t_dst = c.t_dst.copy()
    t_dst[:, [2, 3]] = -1
    dst = random_fill(PagedCache(geom.n_layers, n + 2, c.stride, DEV), 3)
    hk0, hv0 = host_layers(dst)
    vo = check_restore(c, [bytes(r) for r in recs], store2.ptrs, store2.lens, t_dst, dst, hk0, hv0)
    assert vo == [ref.ACCEPT, ref.SEGMENT] + [ref.ACCEPT] * (n - 2)


# Numbers and sizes of blocks on both sides of what one workgroup restores: 192
# KiB with any number, 256 KiB up to 32 blocks, more from 256 blocks on.
@pytest.mark.parametrize("rows,n", [(24, 33), (25, 32), (25, 33), (32, 32), (32, 33), (33, 32), (33, 255), (33, 256)])
def test_blocks_around_one_workgroup(rows, n):
    geom = wl.Geometry(4, 2, 256, rows)  # 8 chunks of `rows` KiB
    c = Case(geom, n, n, n + 2, seed=33)
    c.make_src()
    store, _ = c.save()
    recs = [bytearray(r.tobytes()) for r in store.buf.cpu().numpy()]
    recs[0][c.lay.payload_offset + 5] ^= 1
    recs[n - 2][80] ^= 0x40
    recs[n - 1][-1] ^= 0x40
    store2 = upload_records(recs, c.lay.record_bytes)
    dst = random_fill(PagedCache(geom.n_layers, n + 2, c.stride, DEV), 3)
    hk0, hv0 = host_layers(dst)
    log("around one workgroup", c.lay.record_bytes, "bytes,", n, "blocks")
    vo = check_restore(c, [bytes(r) for r in recs], store2.ptrs, store2.lens, c.t_dst, dst, hk0, hv0)
    assert vo == [ref.SEGMENT] + [ref.ACCEPT] * (n - 3) + [ref.ROOT, ref.SEGMENT]


# Metadata of several tiles (9,984 bytes, the token ids from 5,056 on), which a
# load of 5 blocks waits for and one of 80 does not: the two forms of the checks
# stage it 1 KiB and 4 KiB at a time. Flips on both sides of tile boundaries,
# with the stored root and with one that fits them.
@pytest.mark.parametrize("n", [5, 80])
@pytest.mark.parametrize("offs,reroot", [((1023, 1024, 4095, 4096), False), ((5056, 8191, 8192, 9855), True),
                                         ((9856, 9983, 5055, 6145), True)])
def test_metadata_of_several_tiles(n, offs, reroot):
    geom = wl.Geometry(2, 1, 64, 8, pages_per_block=150)
    c = Case(geom, n, n * 150, n * 150 + 3, seed=37)
    lay = c.lay
    assert (ref.HEADER_BYTES + 8 * lay.n_segments, lay.payload_offset) == (5056, 9984)
    c.make_src()
    store, st = c.save()
    assert (st == ref.ACCEPT).all()
    recs = [bytearray(r.tobytes()) for r in store.buf.cpu().numpy()]
    for b, o in enumerate(offs):
        recs[b][o] ^= 0x04
        if reroot:
            recs[b][144:152] = ref.root_digest(bytes(recs[b][:144]) + bytes(8) + bytes(recs[b][152:9984])).to_bytes(8, "little")
    store2 = upload_records(recs, lay.record_bytes)
    dst = random_fill(PagedCache(geom.n_layers, n * 150 + 3, c.stride, DEV), 3)
    hk0, hv0 = host_layers(dst)
    log("metadata of several tiles", n, "blocks, flips at", offs)
    vo = check_restore(c, [bytes(r) for r in recs], store2.ptrs, store2.lens, c.t_dst, dst, hk0, hv0)
    want = [ref.ROOT] * 4
    if reroot:  # token ids, padding, a chunk digest
        want = [ref.TOKENS if 5056 <= o < 9856 else ref.HEADER if o >= 9856 else ref.SEGMENT for o in offs]
    assert vo[:4] == want and set(vo[4:]) == {ref.ACCEPT}
