"""Host logic of the prefill launch (emm_prefill_plan_host): how a batch is dealt to the XCDs, how many work
units each gets, and how the units left over after full rounds are cut.  What carries weight here are the
invariants the kernels rely on (every unit appears once; the extra workgroups, the workspace records and the
merge workgroups suffice; the workspace size covers any plan the scalar fields admit); the second writing-out of
the rule in plain Python only guards against the C++ and the description drifting apart.  No GPU."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest

from paper_2507_10069_amd import binding as B
from paper_2507_10069_amd import workloads as W

XCDS, CUS, ROWS = 8, 32, 256


def _batch(H, Hkv, new, dtype="bf16", d=128):
    return B.make_batch(num_reqs=len(new), num_q_heads=H, num_kv_heads=Hkv, head_dim=d, page_size=16, num_pages=1 << 20,
                        max_pages_per_req=1 << 16, total_new_tokens=int(sum(new)), max_new_len=int(max(new)) if len(new) else 0,
                        dtype=dtype, softmax_scale=0.1)


def _model(H, Hkv, new):
    """Units per XCD and pieces per left-over unit, from the description of the scheme alone."""
    G = H // Hkv
    pairs = len(new) * Hkv
    fan = 1
    while fan < XCDS and pairs * fan * 2 <= XCDS:
        fan *= 2
    if len(set(new)) > 1:                                      # requests of different lengths: every request on every XCD
        while fan < XCDS and (Hkv * fan) % XCDS:
            fan *= 2
    tiles_of = [-(-new[p // Hkv] * G // ROWS) for p in range(pairs)]
    uniform = len(set(new)) == 1
    cutting = -(-pairs * fan // XCDS) <= 64
    dealt = [0] * XCDS                                         # sub-pair j of pair p has row tiles j, j + fan, ...
    for p in range(pairs):
        for j in range(fan):
            dealt[(p * fan + j) % XCDS] += len(range(j, tiles_of[p], fan))
    units = dealt
    if cutting:                                                # the fan XCDs that share pairs take all their row tiles in turns
        units = []
        for x in range(XCDS):
            first, turn = x - x % fan, x % fan
            listed = sum(tiles_of[sp // fan] for sp in range(first, pairs * fan, XCDS))
            units.append(len(range(turn, listed, fan)))        # (of a single one, two XCDs do a half of the rows each)
    uneven_ok = not (uniform and len(set(dealt)) == 1)
    pieces, ks, halves = [], [], []
    for u in units:
        rem, full = u % CUS, u // CUS
        k = -(-rem // (CUS - rem)) if (16 < rem <= 30 and uneven_ok) else 0
        half = full > 0 and 12 < rem <= 16
        if rem == 0:
            p = 1
        elif k or half:
            p = 2
        elif full == 0:
            p = 1
            while p < 32 and 2 * p * rem <= CUS:
                p *= 2
        else:
            p = 1 if rem > 12 else 2 if rem > 8 else 4
        pieces.append(p); ks.append(k); halves.append(int(half))
    if uniform and cutting and all(p == 1 for p in pieces):
        cutting = False                                        # the host knows that nothing will be cut
    if not cutting:
        pieces, ks, halves = [1] * XCDS, [0] * XCDS, [0] * XCDS
    return fan, units, pieces, ks, halves, cutting


def test_named_workloads():
    cfg3 = W.config(3)
    p = B.emm_prefill_plan_host(_batch(28, 4, cfg3.new_lens.tolist()), cfg3.new_lens)
    assert p["units"] == [56] * 8 and p["cutting"] == 0 and p["grid"] == 448          # two rounds, the second of 24: not cut
    one = B.emm_prefill_plan_host(_batch(28, 4, [36]), [36])                            # a lone unit on every other XCD
    assert one["fan"] == 2 and one["units"] == [1, 0] * 4 and one["pieces"] == [32, 1] * 4 and one["grid"] == 8 * (1 + 31)
    cfg5 = W.config(5)
    p5 = B.emm_prefill_plan_host(_batch(32, 8, cfg5.new_lens.tolist()), cfg5.new_lens)
    want = sum(-(-int(n) * 4 // ROWS) for n in cfg5.new_lens)                           # every XCD holds one KV head of every request
    assert p5["units"] == [want] * 8 and p5["cutting"] == 1
    cfg2 = W.config(2)                                           # requests of different lengths on 4 KV heads: each pair is
    p2 = B.emm_prefill_plan_host(_batch(28, 4, cfg2.new_lens.tolist()), cfg2.new_lens)   # dealt to 2 XCDs, so that every XCD
    assert p2["fan"] == 2                                        # gets half the row tiles of one KV head of every request
    assert max(p2["units"]) - min(p2["units"]) <= 1, p2["units"]
    no_ws = B.emm_prefill_plan_host(_batch(28, 4, [36]), [36], with_workspace=False)
    assert no_ws["cutting"] == 0 and no_ws["pieces"] == [1] * 8 and no_ws["grid"] == 8


@pytest.mark.parametrize("seed", range(40))
def test_random_batches_match_model_and_keep_invariants(seed):
    rng = np.random.default_rng(300 + seed)
    Hkv = int(rng.choice([1, 2, 4, 8, 16]))
    G = int(rng.choice([1, 2, 4, 7, 8]))
    n_req = int(rng.choice([1, 1, 2, 3, 5, 8, 16, 33, 70]))
    top = int(rng.choice([1, 3, 40, 300, 2100]))
    new = [int(x) for x in rng.integers(0, top + 1, n_req)]
    if rng.random() < 0.25:
        new = [top] * n_req                                    # a uniform batch
    if sum(new) == 0:
        new[0] = top
    H = Hkv * G
    p = B.emm_prefill_plan_host(_batch(H, Hkv, new), new)
    fan, units, pieces, ks, halves, cutting = _model(H, Hkv, new)
    assert (p["fan"], p["units"], p["cutting"]) == (fan, units, int(cutting)), (new, p)
    assert (p["pieces"], p["uneven_k"], p["rows_only"]) == (pieces, ks, halves), (new, p)
    assert sum(p["units"]) == sum(-(-n * G // ROWS) for n in new) * Hkv              # every row tile of every pair, once
    assert p["grid"] == XCDS * (p["slots_per_xcd"] + (31 if p["cutting"] else 0))
    if cutting:                                                                        # XCDs that share a list differ by one unit
        assert all(max(p["units"][x:x + fan]) - min(p["units"][x:x + fan]) <= 1 for x in range(0, XCDS, fan)), (new, p)
    for x in range(XCDS):
        rem = p["units"][x] % CUS
        assert p["units"][x] <= p["slots_per_xcd"]                                     # a slot for every unit
        if cutting and fan > 1 and sum(p["units"][x - x % fan:][:fan]) == 1:           # a single unit: row halves on two XCDs
            assert p["slots_per_xcd"] >= 1 and p["units"][x] == int(x % fan == 0)
        assert rem * (p["pieces"][x] - 1) <= 31                                        # extra workgroups for pieces 1, 2, ...
        assert rem * p["pieces"][x] <= 64                                              # workspace slots of the XCD
        shares = 1 if p["uneven_k"][x] else p["pieces"][x]
        assert p["pieces"][x] == 1 or rem * shares <= 32                               # merge workgroups of the XCD
        assert (p["uneven_k"][x] > 0) <= (16 < rem <= 30)


PIECE_BYTES = 66 * 512 * 4          # a piece record: 64 accumulator values, reference exponent and row sum per thread


@pytest.mark.parametrize("seed", range(40))
def test_workspace_size_covers_the_plan(seed):
    """emm_prefill_attn_workspace_size, which sees only the scalar fields, against what the plan for the real lengths
    needs: 8 XCDs x (left-over units x planned pieces) records, laid out with one stride for all XCDs.  It must cover
    the plan for any lengths the scalars admit, be exact when the host can know the plan (all requests alike), and
    be zero when nothing can be cut."""
    rng = np.random.default_rng(900 + seed)
    Hkv = int(rng.choice([1, 2, 4, 8]))
    G = int(rng.choice([1, 4, 7, 8]))
    n_req = int(rng.choice([1, 2, 3, 8, 16, 40]))
    top = int(rng.choice([3, 40, 300, 2100]))
    uniform = rng.random() < 0.4
    new = [top] * n_req if uniform else [int(x) for x in rng.integers(0, top + 1, n_req)]
    if sum(new) == 0:
        new[0] = top
    max_pages = int(rng.choice([16, 64, 600, 4096]))          # contexts of at most 256 .. 65536 tokens
    b = B.make_batch(num_reqs=n_req, num_q_heads=Hkv * G, num_kv_heads=Hkv, head_dim=128, page_size=16, num_pages=1 << 20,
                     max_pages_per_req=max_pages, total_new_tokens=int(sum(new)), max_new_len=int(max(new)), dtype="bf16",
                     softmax_scale=0.1)
    size = B.emm_prefill_attn_workspace_size(b)
    p = B.emm_prefill_plan_host(b, new)
    assert size % (XCDS * PIECE_BYTES) == 0
    stride = size // (XCDS * PIECE_BYTES)                      # records per XCD
    cuttable = max_pages * 16 >= 24 * 64                       # a context of 24 key tiles: the shortest that is ever cut
    need = 0
    for x in range(XCDS):
        rem = p["units"][x] % CUS
        if p["cutting"] and p["pieces"][x] > 1 and not p["rows_only"][x] and cuttable:
            need = max(need, rem * p["pieces"][x])
    assert stride >= need, (new, p, stride)
    if not cuttable or not p["cutting"]:
        assert size == 0
    if len(set(new)) == 1:
        assert stride == need                                   # the host knows every XCD's unit count
    assert stride <= 64


@pytest.mark.parametrize("seed", range(40))
def test_lengths_that_contradict_the_scalars_leave_no_record_outside_the_workspace(seed):
    """The workspace is sized from the scalar fields, the kernels plan from the lengths in device memory.  Whatever those
    hold, the plan cuts along the keys only where an XCD's records fit its share of the workspace."""
    rng = np.random.default_rng(1700 + seed)
    Hkv = int(rng.choice([1, 2, 4, 8]))
    G = int(rng.choice([1, 4, 7, 8]))
    n_req = int(rng.choice([2, 3, 8, 16, 40]))
    top = int(rng.choice([3, 40, 300, 2100]))
    b = _batch(Hkv * G, Hkv, [top] * n_req)                   # the scalars of a uniform batch: the size is exactly its plan's
    stride = B.emm_prefill_attn_workspace_size(b) // (XCDS * PIECE_BYTES)
    for _ in range(20):
        lens = [int(x) for x in rng.integers(-2, top + 40, n_req)]
        p = B.emm_prefill_plan_host(b, lens)
        for x in range(XCDS):
            rem = p["units"][x] % CUS
            if p["cutting"] and p["pieces"][x] > 1 and not p["rows_only"][x]:
                assert rem * p["pieces"][x] <= stride, (lens, p, stride)


def test_workspace_of_the_headline_workload_is_empty():
    cfg3 = W.config(3)
    b = _batch(28, 4, cfg3.new_lens.tolist())
    assert B.emm_prefill_attn_workspace_size(b) == 0          # 56 units per XCD, none cut: no records, no merge


def test_argument_errors():
    lib = B.load()
    plan = B.emm_prefill_plan()
    ok = (ctypes.c_int32 * 2)(5, 5)
    assert lib.emm_prefill_plan_host(None, ok, 1, ctypes.byref(plan)) == B.EMM_ERR_NULL
    b = _batch(8, 2, [5, 5])
    assert lib.emm_prefill_plan_host(ctypes.byref(b), None, 1, ctypes.byref(plan)) == B.EMM_ERR_NULL
    assert lib.emm_prefill_plan_host(ctypes.byref(b), ok, 1, None) == B.EMM_ERR_NULL
    f32 = _batch(8, 2, [5, 5], dtype="f32", d=64)
    assert lib.emm_prefill_plan_host(ctypes.byref(f32), ok, 1, ctypes.byref(plan)) == B.EMM_ERR_UNSUPPORTED
    empty = _batch(8, 2, [])
    assert lib.emm_prefill_plan_host(ctypes.byref(empty), None, 1, ctypes.byref(plan)) == B.EMM_OK and plan.grid == 0


@pytest.mark.parametrize("n_req,Hkv,G,max_pages", [(1, 4, 7, 1024), (8, 4, 7, 1152), (64, 4, 7, 512), (32, 8, 4, 290), (3, 1, 16, 40),
                                                   (200, 8, 1, 64), (1, 4, 7, 8192), (5, 2, 3, 1)])
def test_decode_workspace_holds_the_pieces_of_the_longest_context(n_req, Hkv, G, max_pages):
    """A decode batch's workspace is [pair][piece][16 rows][130 floats]; pieces are 4 .. 124 tiles of 32 keys, and
    there must be enough of them for a context that fills the page-table row."""
    b = B.make_batch(num_reqs=n_req, num_q_heads=Hkv * G, num_kv_heads=Hkv, head_dim=128, page_size=16, num_pages=1 << 20,
                     max_pages_per_req=max_pages, total_new_tokens=n_req, max_new_len=1, dtype="bf16", softmax_scale=0.1)
    per_piece = 16 * 130 * 4
    size = B.emm_prefill_attn_workspace_size(b)
    assert size % (n_req * Hkv * per_piece) == 0
    pieces = size // (n_req * Hkv * per_piece)
    tiles = -(-max_pages * 16 // 32)
    assert -(-tiles // 124) <= pieces <= max(-(-tiles // 4), 1)
    # hints can only shrink it; a hint larger than the table changes nothing
    small = B.make_shared_prefix(0, planned_tiles=n_req * 4, max_own_tiles=4)
    assert B.emm_decode_attn_shared_workspace_size(b, small) <= size
    wide = B.make_shared_prefix(0, planned_tiles=0, max_own_tiles=10 * tiles)
    assert B.emm_decode_attn_shared_workspace_size(b, wide) == size


def test_decode_plan_of_a_single_request_uses_fewer_longer_pieces():
    """One request cannot be ragged: its contexts are cut so that about 1.5 workgroups per compute unit (at most 384)
    stream them, where a batch of several requests is planned for rounds of 512 (and reserves room for shorter pieces)."""
    per_piece = 16 * 130 * 4
    def pieces(n_req, max_pages):
        b = B.make_batch(num_reqs=n_req, num_q_heads=28, num_kv_heads=4, head_dim=128, page_size=16, num_pages=1 << 20,
                         max_pages_per_req=max_pages, total_new_tokens=n_req, max_new_len=1, dtype="bf16", softmax_scale=0.1)
        size = B.emm_prefill_attn_workspace_size(b)
        assert size % (n_req * 4 * per_piece) == 0
        return size // (n_req * 4 * per_piece)
    one = pieces(1, 8192)                                       # 131072 tokens: 4096 tiles of 32 keys per KV head
    assert 256 < 4 * one <= 384
    two = pieces(2, 4096)                                       # the same number of tiles in two requests
    assert 384 < 8 * two <= 768


class _BatchView(ctypes.Structure):
    _fields_ = [(n, ctypes.c_void_p) for n in ("page_table", "prefix_lens", "new_lens", "cu_new_lens")] + \
               [(n, ctypes.c_int32) for n in ("num_reqs", "num_q_heads", "num_kv_heads", "head_dim", "page_size", "num_pages", "max_pages",
                                              "total_new_tokens", "max_new_len", "page_shift")] + [("softmax_scale", ctypes.c_float)]


class _SharedPrefixView(ctypes.Structure):
    _fields_ = [(n, ctypes.c_void_p) for n in ("unit_first_req", "unit_num_reqs", "unit_shared_len", "req_unit", "req_shared_len")] + \
               [(n, ctypes.c_int32) for n in ("num_units", "planned_tiles", "max_own_tiles", "max_unit_tiles")]


class _DecodeShape(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in ("n_pairs", "n_unit_pairs", "tiles_per_piece", "pieces_max", "pieces_unit", "ahead", "late", "stream")]


def _decode_plan(n_req, H, Hkv, table_tokens, planned_tiles=0, max_own_tiles=0, num_units=0, max_unit_tiles=0):
    """The plan of a decode batch, from the library's own planner (emm::attn_bf16_decode_shape)."""
    plan = B.load()["_ZN3emm22attn_bf16_decode_shapeERKNS_9BatchViewERKNS_16SharedPrefixViewE"]
    plan.restype = _DecodeShape
    plan.argtypes = [ctypes.POINTER(_BatchView), ctypes.POINTER(_SharedPrefixView)]
    b = _BatchView(num_reqs=n_req, num_q_heads=H, num_kv_heads=Hkv, head_dim=128, page_size=16, num_pages=1 << 20,
                   max_pages=-(-table_tokens // 16), total_new_tokens=n_req, max_new_len=1, softmax_scale=0.1)
    return plan(b, _SharedPrefixView(num_units=num_units, planned_tiles=planned_tiles, max_own_tiles=max_own_tiles, max_unit_tiles=max_unit_tiles))


def test_decode_streams_by_what_is_known_of_the_work():
    """More than 96 MiB of K and V are fetched past the caches.  The width of the page table says how long the contexts may be,
    not how long they are: without the amount of work each workgroup decides by the length of its own context."""
    NEVER, PRIVATE, BY_LENGTHS = 0, 1, 2
    assert _decode_plan(1, 28, 4, 131072).stream == BY_LENGTHS                 # a chat of whatever length behind a wide row
    assert _decode_plan(64, 28, 4, 8192).stream == BY_LENGTHS
    assert _decode_plan(1, 28, 4, 40000).stream == NEVER                       # 82 MB at most
    assert _decode_plan(1, 28, 4, 131072, planned_tiles=47, max_own_tiles=47).stream == NEVER
    assert _decode_plan(64, 28, 4, 8192, planned_tiles=64 * 256, max_own_tiles=256).stream == PRIVATE
    assert _decode_plan(64, 28, 4, 8192, planned_tiles=64 * 23, max_own_tiles=256).stream == NEVER


def test_decode_merge_asks_ahead_only_for_what_is_there():
    """The merge kernel may ask for records before it knows the lengths where those are few or most of them exist."""
    assert _decode_plan(1, 28, 4, 1504).ahead == 1                             # 28 rows of 12 records
    assert _decode_plan(64, 28, 4, 131072).ahead == 0                          # up to 1792 rows of 32 records, who knows how many of them
    assert _decode_plan(64, 28, 4, 131072, planned_tiles=64 * 4096, max_own_tiles=4096).ahead == 1
    assert _decode_plan(64, 28, 4, 131072, planned_tiles=64 * 40, max_own_tiles=4096).ahead == 0      # one long context, the others short


# piece lengths (tiles of 32 keys) that measured within 10 % of the best for batches whose contexts are spread evenly
@pytest.mark.parametrize("n_req,H,Hkv,lo,hi,shortest,longest", [(25, 28, 4, 800, 8000, 16, 45), (19, 28, 4, 800, 8000, 22, 36), (12, 28, 4, 800, 8000, 16, 28),
                                                                (19, 32, 8, 384, 3844, 24, 36), (74, 16, 2, 401, 4019, 26, 36)])
def test_decode_plan_of_contexts_known_to_differ(n_req, H, Hkv, lo, hi, shortest, longest):
    """With the amount of work given, a batch whose contexts differ is not cut in pieces so long that a compute unit which gets
    two of them ends long after the others."""
    tiles = [-(-int(c) // 32) for c in np.linspace(lo, hi, n_req)]
    S = _decode_plan(n_req, H, Hkv, hi, planned_tiles=sum(tiles), max_own_tiles=max(tiles))
    assert shortest <= S.tiles_per_piece <= longest, S.tiles_per_piece
    assert S.pieces_max == -(-max(tiles) // S.tiles_per_piece)


@pytest.mark.parametrize("n_req,H,Hkv,tokens,pairs", [(8, 28, 4, 900, True), (16, 28, 4, 400, True), (8, 28, 4, 1024, True), (8, 28, 4, 1025, False),
                                                      (5, 32, 8, 720, True), (1, 32, 8, 3889, True), (1, 32, 8, 4097, False)])
def test_decode_plan_takes_pieces_of_two_blocks_a_wave_while_each_has_a_compute_unit(n_req, H, Hkv, tokens, pairs):
    """Pieces of four tiles are the quickest as long as there are at most 256 of them in all; from 257 on longer ones are."""
    tiles = -(-tokens // 32)
    S = _decode_plan(n_req, H, Hkv, 32 * tiles, planned_tiles=n_req * tiles, max_own_tiles=tiles)
    assert (S.tiles_per_piece == 4) == pairs, S.tiles_per_piece


@pytest.mark.parametrize("n_req,H,Hkv,tokens,hint", [(1, 28, 4, 300, False), (1, 32, 4, 320, False), (8, 40, 8, 300, False), (1, 64, 8, 320, True), (8, 28, 4, 320, True), (64, 8, 1, 317, False)])
def test_decode_plan_of_ten_tiles_is_one_piece(n_req, H, Hkv, tokens, hint):
    """What pieces of two blocks a wave save does not make up for the merge of so short a context."""
    tiles = -(-tokens // 32)
    S = _decode_plan(n_req, H, Hkv, 32 * tiles, **(dict(planned_tiles=n_req * tiles, max_own_tiles=tiles) if hint else {}))
    assert S.pieces_max == 1, S.tiles_per_piece


def _plan_of_units(H, Hkv, units, private):
    """The plan of a batch of units (members, shared tokens, own tokens of each) and private contexts (requests, tokens), told all there is to tell."""
    tiles = lambda tokens: -(-tokens // 32)
    planned = sum(shared // 32 + n * tiles(own) for n, shared, own in units) + sum(n * tiles(tokens) for n, tokens in private)
    return _decode_plan(sum(n for n, _, _ in units) + sum(n for n, _ in private), H, Hkv, max([s + o for _, s, o in units] + [t for _, t in private]), planned_tiles=planned,
                        max_own_tiles=max([tiles(o) for _, _, o in units] + [tiles(t) for _, t in private]), num_units=len(units),
                        max_unit_tiles=max(s // 32 for _, s, _ in units))


# groups beside private chats, which one by one would all be planned as long as the longest; large groups of one query head per KV head, whose members
# would read the shared keys 32 times
@pytest.mark.parametrize("H,Hkv,units,private", [(28, 4, [(2, 6016, 60)], [(40, 100)]), (28, 4, [(2, 3008, 60)], [(30, 200)]), (32, 8, [(2, 2048, 60)], [(60, 60)]),
                                                 (8, 8, [(32, 2048, 60)], []), (8, 8, [(32, 1984, 20)] * 2, []), (2, 2, [(32, 6400, 20)] * 2, []), (16, 8, [(7, 2048, 90), (4, 128, 90)], [])])
def test_decode_plan_keeps_units_that_save_reading(H, Hkv, units, private):
    S = _plan_of_units(H, Hkv, units, private)
    assert S.n_unit_pairs == len(units) * Hkv
    assert S.tiles_per_piece <= 10


@pytest.mark.parametrize("H,Hkv,units,private", [(28, 4, [(3, 2432, 100)], []), (28, 4, [(4, 1856, 100)] * 2, []), (32, 8, [(5, 1856, 60)] * 2, []), (32, 8, [(4, 1024, 60)], [(1, 90)]),
                                                 (2, 2, [(16, 1536, 100), (3, 704, 100)], [(1, 100)]), (28, 4, [(3, 2816, 100), (4, 96, 100), (2, 1216, 100), (3, 672, 100)], [(4, 500)]),
                                                 (32, 8, [(8, 992, 60)], [(8, 500)])])
def test_decode_plan_leaves_units_aside_where_there_is_little_to_read(H, Hkv, units, private):
    S = _plan_of_units(H, Hkv, units, private)
    assert S.n_unit_pairs == 0 and S.pieces_unit <= 1
    assert S.stream == 0 and S.late == 0                     # as the amount of work has it: all fits the caches


@pytest.mark.parametrize("seed", range(20))
def test_decode_plan_of_equal_contexts_is_cut_evenly(seed):
    """Pieces of equal contexts are as short as their number allows: no last piece that is a sliver beside the others."""
    rng = np.random.default_rng(2100 + seed)
    for _ in range(20):
        Hkv, n_req = int(rng.choice([1, 2, 4, 8])), int(rng.choice([1, 2, 5, 16, 64, 100]))
        tiles = int(2 ** rng.uniform(3, 11))
        if Hkv * n_req * -(-tiles // 124) > 2016:
            continue
        hints = dict(planned_tiles=n_req * tiles, max_own_tiles=tiles) if rng.random() < 0.5 else {}
        S = _decode_plan(n_req, 4 * Hkv, Hkv, 32 * tiles, **hints)
        assert S.pieces_max == -(-tiles // S.tiles_per_piece)
        assert S.tiles_per_piece == 4 or -(-tiles // (S.tiles_per_piece - 1)) > S.pieces_max, (n_req, Hkv, tiles, S.tiles_per_piece)


# piece lengths that measured within 8 % of the best for contexts spread from a quarter of this length up, and for equal ones
@pytest.mark.parametrize("n_req,H,Hkv,longest,shortest_piece,longest_piece", [(22, 32, 8, 4880, 36, 46), (40, 28, 4, 4000, 42, 45), (64, 28, 4, 8191, 43, 86),
                                                                              (8, 28, 4, 18000, 24, 44), (128, 28, 4, 1000, 32, 32)])
def test_decode_plan_without_hints_suits_equal_and_different_contexts(n_req, H, Hkv, longest, shortest_piece, longest_piece):
    S = _decode_plan(n_req, H, Hkv, longest)
    assert shortest_piece <= S.tiles_per_piece <= longest_piece, S.tiles_per_piece


@pytest.mark.parametrize("seed", range(20))
def test_decode_hints_never_grow_the_workspace(seed):
    """Whatever hints a step brings, the workspace that the batch without hints asks for is enough (no units)."""
    rng = np.random.default_rng(2300 + seed)
    for _ in range(50):
        Hkv, G, n_req = int(rng.choice([1, 2, 4, 8])), int(rng.choice([1, 4, 7, 8])), int(rng.integers(1, 65))
        top = int(2 ** rng.uniform(6, 16))
        ctx = rng.integers(1, top + 1, n_req)
        width = int(-(-int(ctx.max()) // 16) * rng.choice([1, 1, 2, 8]))
        b = B.make_batch(num_reqs=n_req, num_q_heads=Hkv * G, num_kv_heads=Hkv, head_dim=128, page_size=16, num_pages=1 << 20,
                         max_pages_per_req=width, total_new_tokens=n_req, max_new_len=1, dtype="bf16", softmax_scale=0.1)
        size = B.emm_prefill_attn_workspace_size(b)
        tiles = -(-ctx // 32)
        for hints in ({"planned_tiles": int(tiles.sum()), "max_own_tiles": int(tiles.max())}, {"planned_tiles": int(tiles.sum())},
                      {"max_own_tiles": int(tiles.max())}, {"planned_tiles": int(rng.integers(1, 2 * n_req * top))}):
            assert B.emm_decode_attn_shared_workspace_size(b, B.make_shared_prefix(0, **hints)) <= size, (n_req, Hkv, width, hints)
        assert B.emm_decode_attn_shared_workspace_size(b, B.make_shared_prefix(0)) == size
        assert B.emm_decode_attn_shared_workspace_size(b, B.make_shared_prefix(0, max_unit_tiles=3)) == size


def test_decode_workgroups_leave_on_the_lengths_where_most_have_no_work():
    """Page ids are asked for together with the lengths unless the grid is that of a table much wider than the chip needs."""
    assert _decode_plan(64, 28, 4, 131072).late == 1 and _decode_plan(256, 32, 8, 131072).late == 1
    assert _decode_plan(64, 28, 4, 8192).late == 0 and _decode_plan(1, 28, 4, 131072).late == 0
    assert _decode_plan(64, 28, 4, 131072, planned_tiles=64 * 47, max_own_tiles=50).late == 0
