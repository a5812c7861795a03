"""GPU parity of the fused QKV projection with its rotary / cache epilogue (oppo_qkv_proj_rope_append)
against the float64 oracle (oracle/projection.py), and of the layer path projection -> attention
against the oracle's projection -> rotation -> one-shot prefill.

Tolerance of the projection: the kernel accumulates bf16 products in fp32 (MFMA), rotates in fp32 and
rounds once to bf16, so |gpu - oracle| <= 2^-8 |oracle| (half a bf16 ulp at most) plus the fp32
accumulation and rotation error, bounded by 2^-19 * sum_k |x_k| |w_k| of the columns involved: a sum over
hidden takes N = hidden / 16 matrix instructions, each rounding a partial sum to within 2^-24 of itself; those of
independent N(0, 1) terms stay below ~4.5 sqrt(16 i) against 10 N of the sum of magnitudes, so that even roundings
which all point one way come to 1.2 sqrt(N) 2^-24 of it: 17 * 2^-24 at hidden 3072, the longest here, of 32 * 2^-24.
Keys and values are compared where they land: in the cache, whose other slots must stay untouched."""
import ctypes

import numpy as np
import pytest

from oracle import bf16_bits_to_f64, full_prefill, pass_positions, qkv_projection, qkv_projection_rope
from paper_2509_25762_amd.workload import f32_to_bf16_bits

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_25762_amd import binding
    binding.load()
    return binding, torch


def draw(rng, shape, scale=1.0):
    return f32_to_bf16_bits((rng.standard_normal(shape) * scale).astype(np.float32))


def run_projection(gpu, rng, Hq, Hkv, D, hidden, kv_before, q_len, base):
    binding, torch = gpu
    dev = torch.device("cuda:0")
    B = len(q_len)
    cu = np.concatenate([[0], np.cumsum(q_len)]).astype(np.int32)
    rows = int(cu[-1])
    xb = draw(rng, (rows, hidden))
    wb = draw(rng, ((Hq + 2 * Hkv) * D, hidden), 1.0 / np.sqrt(hidden))
    cap = np.asarray(kv_before, dtype=np.int64) + q_len + 2
    slot_begin = np.concatenate([[0], np.cumsum(cap)])
    ck = torch.full((int(slot_begin[-1]), Hkv, D), -1, dtype=torch.int16, device=dev)
    cv = torch.full_like(ck, -1)
    cache = binding.KVCache(ck, cv, slot_begin, np.asarray(kv_before, dtype=np.int32))
    desc = binding.make_desc(Hq, Hkv, D, 1.0 / np.sqrt(D))
    tx = torch.from_numpy(xb.view(np.int16)).to(dev)
    tw = torch.from_numpy(wb.view(np.int16)).to(dev)
    q_out = torch.full((rows + 2, Hq, D), 0x7FC0, dtype=torch.int16, device=dev)     # a spare row on either side
    ws = torch.empty(binding.oppo_qkv_proj_workspace_bytes(desc, rows), dtype=torch.uint8, device=dev)
    binding.oppo_qkv_proj_rope_append(desc, cache, cu, tx, hidden, tw, q_out[1:-1], ws, base)
    torch.cuda.synchronize()
    return xb, wb, cu, slot_begin, cache, q_out.cpu().numpy().view(np.uint16), ck.cpu().numpy().view(np.uint16), cv.cpu().numpy().view(np.uint16)


def bound_of(want, mag):
    return 2.0 ** -8 * np.abs(want) * 1.001 + 2.0 ** -19 * mag + 1e-30


@pytest.mark.parametrize("Hq,Hkv,D,hidden,base", [(8, 2, 128, 256, 10000.0), (4, 4, 64, 128, 500000.0), (3, 1, 64, 1024, 10000.0),
                                                   (16, 1, 128, 512, 1000000.0), (2, 1, 64, 64, 10000.0)])   # the last: one k tile
def test_projection_epilogue_matches_the_oracle_on_a_ragged_pass(gpu, Hq, Hkv, D, hidden, base):
    rng = np.random.default_rng(300 + Hq + D + hidden)
    q_len = np.array([0, 1, 7, 64, 130, 9, 0, 33, 129], dtype=np.int32)          # 373 rows: three row tiles, a ragged last one
    kv_before = np.array([17, 0, 60000, 123, 4095, 1, 5, 65536 * 4, 3], dtype=np.int32)
    xb, wb, cu, slot_begin, cache, gq, gk, gv = run_projection(gpu, rng, Hq, Hkv, D, hidden, kv_before, q_len, base)
    pos = pass_positions(kv_before, q_len)
    q_ref, k_ref, v_ref = qkv_projection_rope(xb, wb, pos, Hq, Hkv, D, base)
    # magnitudes sum_k |x||w| per output column, and per rotated pair
    mag = np.abs(bf16_bits_to_f64(xb)) @ np.abs(bf16_bits_to_f64(wb)).T
    qc, kc = Hq * D, Hkv * D
    half = D // 2

    def pair(m, heads):
        m = m.reshape(m.shape[0], heads, D)
        p = m[..., :half] + m[..., half:]
        return np.concatenate([p, p], axis=-1)

    assert (gq[0] == 0x7FC0).all() and (gq[-1] == 0x7FC0).all(), "rows outside the pass were written"
    got_q = bf16_bits_to_f64(gq[1:-1])
    assert (np.abs(got_q - q_ref) <= bound_of(q_ref, pair(mag[:, :qc], Hq))).all(), "queries"
    assert cache.kv_len.tolist() == (kv_before + q_len).tolist()
    for i in range(len(q_len)):
        b, n0, n1 = int(slot_begin[i]), int(kv_before[i]), int(kv_before[i] + q_len[i])
        r0, r1 = int(cu[i]), int(cu[i + 1])
        got_k, got_v = bf16_bits_to_f64(gk[b + n0:b + n1]), bf16_bits_to_f64(gv[b + n0:b + n1])
        assert (np.abs(got_k - k_ref[r0:r1]) <= bound_of(k_ref[r0:r1], pair(mag[r0:r1, qc:qc + kc], Hkv))).all(), f"keys of sequence {i}"
        assert (np.abs(got_v - v_ref[r0:r1]) <= bound_of(v_ref[r0:r1], mag[r0:r1, qc + kc:].reshape(r1 - r0, Hkv, D))).all(), f"values of sequence {i}"
        # slots before and after the appended rows are untouched
        assert (gk[b:b + n0] == 0xFFFF).all() and (gk[b + n1:int(slot_begin[i + 1])] == 0xFFFF).all()
        assert (gv[b:b + n0] == 0xFFFF).all() and (gv[b + n1:int(slot_begin[i + 1])] == 0xFFFF).all()
    # almost every element is the oracle's value rounded to bf16 (fp32 noise crosses a rounding boundary rarely)
    differ = int((gq[1:-1] != f32_to_bf16_bits(q_ref.astype(np.float32))).sum())
    assert differ <= max(4, gq[1:-1].size // 200), f"{differ} of {gq[1:-1].size} query elements differ from the rounded oracle value"


@pytest.mark.parametrize("rows", [4091, 8155])
def test_larger_passes_take_the_larger_tiles(gpu, rows):
    """The launch picks the tile height from the pass's size: 64 rows for the thin passes above, 128 rows for
    ~4K rows x 6 column tiles and 256 rows for ~8K (plan_qkv_proj chooses); both with a ragged last
    row tile and sequences of uneven length, against the oracle as above."""
    Hq, Hkv, D, hidden, base = 8, 2, 128, 256, 10000.0
    rng = np.random.default_rng(900 + rows)
    q_len = np.array([rows // 2, 1, rows // 4 + 3, 0, 517], dtype=np.int32)
    q_len = np.append(q_len, rows - q_len.sum()).astype(np.int32)
    assert (q_len >= 0).all() and q_len.sum() == rows
    kv_before = np.array([3, 70000, 0, 9, 255, 1024], dtype=np.int32)
    xb, wb, cu, slot_begin, cache, gq, gk, gv = run_projection(gpu, rng, Hq, Hkv, D, hidden, kv_before, q_len, base)
    q_ref, k_ref, v_ref = qkv_projection_rope(xb, wb, pass_positions(kv_before, q_len), Hq, Hkv, D, base)
    mag = np.abs(bf16_bits_to_f64(xb)) @ np.abs(bf16_bits_to_f64(wb)).T
    qc, kc, half = Hq * D, Hkv * D, D // 2

    def pair(m, heads):
        m = m.reshape(m.shape[0], heads, D)
        p = m[..., :half] + m[..., half:]
        return np.concatenate([p, p], axis=-1)

    assert (gq[0] == 0x7FC0).all() and (gq[-1] == 0x7FC0).all(), "rows outside the pass were written"
    assert (np.abs(bf16_bits_to_f64(gq[1:-1]) - q_ref) <= bound_of(q_ref, pair(mag[:, :qc], Hq))).all(), "queries"
    assert cache.kv_len.tolist() == (kv_before + q_len).tolist()
    for i in range(len(q_len)):
        b, n0, n1 = int(slot_begin[i]), int(kv_before[i]), int(kv_before[i] + q_len[i])
        r0, r1 = int(cu[i]), int(cu[i + 1])
        got_k, got_v = bf16_bits_to_f64(gk[b + n0:b + n1]), bf16_bits_to_f64(gv[b + n0:b + n1])
        assert (np.abs(got_k - k_ref[r0:r1]) <= bound_of(k_ref[r0:r1], pair(mag[r0:r1, qc:qc + kc], Hkv))).all(), f"keys of sequence {i}"
        assert (np.abs(got_v - v_ref[r0:r1]) <= bound_of(v_ref[r0:r1], mag[r0:r1, qc + kc:].reshape(r1 - r0, Hkv, D))).all(), f"values of sequence {i}"
        assert (gk[b:b + n0] == 0xFFFF).all() and (gk[b + n1:int(slot_begin[i + 1])] == 0xFFFF).all()
        assert (gv[b:b + n0] == 0xFFFF).all() and (gv[b + n1:int(slot_begin[i + 1])] == 0xFFFF).all()


def check_run(gpu, rng, Hq, Hkv, D, hidden, kv_before, q_len):
    """A pass against the oracle, bounds as above; every other slot and row untouched."""
    rows = int(q_len.sum())
    xb, wb, cu, slot_begin, cache, gq, gk, gv = run_projection(gpu, rng, Hq, Hkv, D, hidden, kv_before, q_len, 10000.0)
    q_ref, k_ref, v_ref = qkv_projection_rope(xb, wb, pass_positions(kv_before, q_len), Hq, Hkv, D, 10000.0)
    mag = (np.abs(bf16_bits_to_f64(xb)) @ np.abs(bf16_bits_to_f64(wb)).T).reshape(rows, Hq + 2 * Hkv, D)
    pair = np.tile(mag[..., :D // 2] + mag[..., D // 2:], 2)
    assert (gq[0] == 0x7FC0).all() and (gq[-1] == 0x7FC0).all(), "rows outside the pass were written"
    assert (np.abs(bf16_bits_to_f64(gq[1:-1]) - q_ref) <= bound_of(q_ref, pair[:, :Hq])).all(), "queries"
    slots = np.concatenate([int(slot_begin[i]) + int(kv_before[i]) + np.arange(q_len[i]) for i in range(len(q_len))])
    assert (np.abs(bf16_bits_to_f64(gk[slots]) - k_ref) <= bound_of(k_ref, pair[:, Hq:Hq + Hkv])).all(), "keys"
    assert (np.abs(bf16_bits_to_f64(gv[slots]) - v_ref) <= bound_of(v_ref, mag[:, Hq + Hkv:])).all(), "values"
    others = np.setdiff1d(np.arange(gk.shape[0]), slots)
    assert (gk[others] == 0xFFFF).all() and (gv[others] == 0xFFFF).all(), "other cache slots were written"


def check_pass(gpu, rows, Hq, Hkv, D, hidden):
    """... of four sequences, one of which sits out."""
    check_run(gpu, np.random.default_rng(rows + hidden), Hq, Hkv, D, hidden, np.array([3, 70000, 0, 9], dtype=np.int32),
              np.array([rows - 1000, 1, 0, 999], dtype=np.int32))


# Passes by the launches they have to take: (rows, Hq, Hkv, D, hidden, [(rows, tile rows, phased, rounds), ..]).
# That the library still cuts them so is asserted here and, without a GPU, in test_boundary_cpu.py.
PASSES = [
    # tiles of 64 and 128 rows
    (6001, 8, 2, 128, 64, [(6001, 64, False, 3)]),           # one k tile, a ragged last row tile
    (6145, 16, 4, 64, 192, [(6145, 64, False, 3)]),          # one row in the last row tile
    (8155, 16, 4, 64, 128, [(8155, 64, False, 3)]),
    (8064, 5, 1, 128, 192, [(8064, 128, False, 1)]),         # a last column tile that is half empty, row tiles without a remainder
    (10789, 8, 2, 128, 128, [(10789, 128, False, 2)]),
    (10789, 8, 2, 128, 1024, [(10789, 128, False, 2)]),      # three stages of the ring, 16 k tiles, two rounds
    # tiles of 256 rows for short k loops
    (27400, 8, 2, 128, 64, [(27400, 256, False, 3)]),        # one k tile, three rounds
    (24600, 5, 1, 128, 128, [(24600, 256, False, 2)]),       # two k tiles, a last column tile that is half empty
    (6800, 16, 4, 64, 320, [(6800, 256, False, 1)]),         # five k tiles, head size 64
    # the phased kernel with tiles of 192 rows: odd and even k tiles, counted waits on every one in the middle
    (5617, 8, 2, 128, 320, [(5617, 192, True, 1)]),
    (6001, 8, 2, 128, 576, [(6001, 192, True, 1)]),
    (5521, 16, 4, 64, 512, [(5521, 192, True, 1)]),
    (16600, 3, 1, 64, 320, [(16600, 192, True, 1)]),         # columns of one whole tile and a quarter
    (8300, 5, 1, 128, 512, [(8300, 192, True, 1)]),          # ... of three and a half
    (11041, 8, 2, 128, 512, [(11041, 192, True, 2)]),        # workgroups with a second tile
    (11041, 16, 4, 64, 576, [(11041, 192, True, 2)]),
    (16600, 5, 1, 128, 512, [(16600, 192, True, 2)]),        # ... and a half-empty column
    # the phased kernel with tiles of 256 rows
    (8155, 8, 2, 128, 1536, [(8155, 256, True, 1)]),
    (8155, 16, 4, 64, 1600, [(8155, 256, True, 1)]),         # 25 k tiles
    (12301, 5, 1, 128, 1536, [(12301, 256, True, 1)]),       # a half-empty column
    (16600, 8, 2, 128, 1536, [(16600, 256, True, 2)]),       # workgroups with a second tile
    (16600, 16, 4, 64, 1600, [(16600, 256, True, 2)]),
    # passes cut into two launches: both heights and both kernels as the second
    (3682, 64, 8, 128, 1536, [(3072, 256, True, 2), (610, 128, False, 1)]),
    (5014, 64, 8, 128, 1536, [(4864, 256, True, 3), (150, 64, False, 1)]),
    (5125, 33, 3, 128, 3072, [(3072, 256, True, 1), (2053, 192, True, 1)]),
    (7937, 65, 5, 64, 1536, [(6656, 256, True, 2), (1281, 128, False, 1)]),
    (5384, 65, 5, 64, 3072, [(3328, 256, True, 1), (2056, 192, True, 1)]),
]


@pytest.mark.parametrize("rows,Hq,Hkv,D,hidden,launches", PASSES)
def test_every_kind_of_tile_and_cut(gpu, rows, Hq, Hkv, D, hidden, launches):
    assert gpu[0].oppo_qkv_proj_plan_debug(gpu[0].make_desc(Hq, Hkv, D, 1.0), rows, hidden) == launches
    check_pass(gpu, rows, Hq, Hkv, D, hidden)


@pytest.mark.parametrize("rows,Hq,Hkv,D,hidden", [(16600, 8, 2, 128, 1536), (11041, 16, 4, 64, 576), (3682, 64, 8, 128, 1536)])
def test_a_stream_confined_to_part_of_the_chip(gpu, rows, Hq, Hkv, D, hidden):
    """On such a stream (here 192 compute units) every tile of the phased kernel has a workgroup of its own instead of one
    that stays for several: the same bits as on an ordinary stream, and as on the default streams (0, 1 and 2: the null,
    legacy and per-thread stream), which are no objects with a mask."""
    binding, torch = gpu
    assert binding.oppo_qkv_proj_plan_debug(binding.make_desc(Hq, Hkv, D, 1.0), rows, hidden)[0][2:] == (True, 2)
    hip = ctypes.CDLL("libamdhip64.so")
    words = (ctypes.c_uint32 * 8)(*([0xFFFFFFFF] * 6 + [0, 0]))
    handle = ctypes.c_void_p()
    if hip.hipExtStreamCreateWithCUMask(ctypes.byref(handle), 8, words) != 0 or not handle.value:
        pytest.skip("no masks of compute units here")
    dev = torch.device("cuda:0")
    x = torch.randn((rows, hidden), device=dev, dtype=torch.bfloat16)
    w = torch.randn(((Hq + 2 * Hkv) * D, hidden), device=dev, dtype=torch.bfloat16) * hidden ** -0.5
    desc = binding.make_desc(Hq, Hkv, D, 1.0)
    got = []
    for stream in (torch.cuda.Stream(), torch.cuda.ExternalStream(handle.value), 0, 1, 2):
        cache = binding.KVCache(torch.zeros((rows, Hkv, D), device=dev, dtype=torch.bfloat16),
                                torch.zeros((rows, Hkv, D), device=dev, dtype=torch.bfloat16), [0, rows])
        q = torch.zeros((rows, Hq, D), device=dev, dtype=torch.bfloat16)
        ws = torch.empty(binding.oppo_qkv_proj_workspace_bytes(desc, rows), dtype=torch.uint8, device=dev)
        torch.cuda.synchronize()
        binding.oppo_qkv_proj_rope_append(desc, cache, [0, rows], x, hidden, w, q, ws, stream=stream)
        torch.cuda.synchronize()
        got.append((q, cache.k, cache.v))
    assert got[0][0].any() and all(torch.equal(a, b) for other in got[1:] for a, b in zip(got[0], other))


@pytest.mark.parametrize("B,Hq,Hkv,D,hidden", [(64, 3, 1, 128, 64), (65, 3, 1, 128, 64), (64, 4, 4, 64, 128), (65, 4, 4, 64, 128),
                                               (1001, 2, 1, 64, 64), (9, 12, 2, 128, 64), (110, 12, 2, 128, 64)])
def test_row_lists_on_either_side_of_their_limits(gpu, B, Hq, Hkv, D, hidden):
    """64 sequences travel in the short list of the row kernel's arguments, 65 in the long one, 1001 in two of them;
    1 .. 9 rows each (the row kernel takes 8 at a time), every third one up to 70,000 tokens in.  The last two: one row
    tile and nine (a group of eight and one of a single tile) by eight column tiles."""
    rng = np.random.default_rng(B + D)
    q_len = (1 + np.arange(B) % 9).astype(np.int32)
    kv_before = ((np.arange(B) * 37) % 50 + (np.arange(B) % 3 == 0) * (70000 if B < 100 else 100)).astype(np.int32)
    check_run(gpu, rng, Hq, Hkv, D, hidden, kv_before, q_len)


@pytest.mark.parametrize("rows,Hq,Hkv,D", [(2048, 3, 1, 128), (2049, 3, 1, 128), (4096, 2, 1, 64), (4097, 2, 1, 64)])
def test_angles_one_by_one_and_in_runs(gpu, rows, Hq, Hkv, D):
    """Up to two waves on every SIMD with a thread per angle each angle has its own sine, beyond that runs of four tokens share
    one.  Runs of every remainder, at positions where the fastest pair has turned thousands of times."""
    q_len = np.array([1, 2, 3, 4, 5, 6, 7, 8, 9, 0, 63, 65, 300], dtype=np.int32)
    q_len = np.append(q_len, rows - q_len.sum()).astype(np.int32)
    kv_before = np.array([0, 65536 * 4, 1, 70001, 17, 2, 90002, 5, 131071, 3, 40003, 8, 0, 20001], dtype=np.int32)
    check_run(gpu, np.random.default_rng(rows), Hq, Hkv, D, 64, kv_before, q_len)


def test_values_are_the_rounded_fp32_sums_when_products_are_exact(gpu):
    """Small integers: every product and partial sum is exact in fp32, so value heads (no rotation) and
    the rows at position 0 (rotation by 0) must be bit-exact, whatever the order of accumulation."""
    binding, torch = gpu
    rng = np.random.default_rng(9)
    Hq, Hkv, D, hidden = 4, 2, 128, 128
    q_len = np.array([200, 1], dtype=np.int32)
    kv_before = np.array([0, 0], dtype=np.int32)
    cu = np.concatenate([[0], np.cumsum(q_len)]).astype(np.int32)
    rows = int(cu[-1])
    xb = f32_to_bf16_bits(rng.integers(-3, 4, size=(rows, hidden)).astype(np.float32))
    wb = f32_to_bf16_bits(rng.integers(-2, 3, size=((Hq + 2 * Hkv) * D, hidden)).astype(np.float32))
    dev = torch.device("cuda:0")
    slot_begin = np.array([0, 200, 201], dtype=np.int64)
    ck = torch.full((201, Hkv, D), -1, dtype=torch.int16, device=dev)
    cv = torch.full_like(ck, -1)
    cache = binding.KVCache(ck, cv, slot_begin, kv_before)
    desc = binding.make_desc(Hq, Hkv, D, 1.0 / np.sqrt(D))
    q_out = torch.zeros((rows, Hq, D), dtype=torch.int16, device=dev)
    ws = torch.empty(binding.oppo_qkv_proj_workspace_bytes(desc, rows), dtype=torch.uint8, device=dev)
    binding.oppo_qkv_proj_rope_append(desc, cache, cu, torch.from_numpy(xb.view(np.int16)).to(dev), hidden,
                                      torch.from_numpy(wb.view(np.int16)).to(dev), q_out, ws)
    torch.cuda.synchronize()
    q_ref, k_ref, v_ref = qkv_projection(xb, wb, Hq, Hkv, D)
    assert np.array_equal(cv.cpu().numpy().view(np.uint16), f32_to_bf16_bits(v_ref.astype(np.float32)))
    gq = q_out.cpu().numpy().view(np.uint16)
    for r in (0, 200):                                   # the two rows at position 0
        assert np.array_equal(gq[r], f32_to_bf16_bits(q_ref[r].astype(np.float32)))
        assert np.array_equal(ck.cpu().numpy().view(np.uint16)[r], f32_to_bf16_bits(k_ref[r].astype(np.float32)))


def test_layer_path_projection_then_attention_equals_one_shot(gpu):
    """Hidden rows streamed in ragged chunks: projection (+ rotation, + cache write) then oppo_chunk_prefill_attn,
    against the oracle's projection -> rotation of all rows -> one-shot prefill, to the attention's tolerance."""
    binding, torch = gpu
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(77)
    Hq, Hkv, D, hidden, base = 8, 2, 128, 256, 10000.0
    n_tok = np.array([150, 40, 300])
    B = len(n_tok)
    xs = [draw(rng, (int(n), hidden)) for n in n_tok]
    wb = draw(rng, ((Hq + 2 * Hkv) * D, hidden), 1.0 / np.sqrt(hidden))
    desc = binding.make_desc(Hq, Hkv, D, 1.0 / np.sqrt(D))
    slot_begin = np.concatenate([[0], np.cumsum(n_tok + 1)])
    ck = torch.full((int(slot_begin[-1]), Hkv, D), -1, dtype=torch.int16, device=dev)
    cv = torch.full_like(ck, -1)
    cache = binding.KVCache(ck, cv, slot_begin)
    tw = torch.from_numpy(wb.view(np.int16)).to(dev)
    outs = [np.zeros((int(n), Hq, D), dtype=np.uint16) for n in n_tok]
    done = np.zeros(B, dtype=np.int64)
    for chunk in ([70, 40, 1], [64, 0, 200], [16, 0, 99]):
        ql = np.array(chunk)
        cu = np.concatenate([[0], np.cumsum(ql)]).astype(np.int32)
        rows = int(cu[-1])
        xb = np.concatenate([xs[i][done[i]:done[i] + ql[i]] for i in range(B)])
        q_rot = torch.empty((rows, Hq, D), dtype=torch.int16, device=dev)
        out = torch.empty_like(q_rot)
        ws = torch.empty(binding.oppo_qkv_proj_workspace_bytes(desc, rows), dtype=torch.uint8, device=dev)
        binding.oppo_qkv_proj_rope_append(desc, cache, cu, torch.from_numpy(xb.view(np.int16)).to(dev), hidden, tw, q_rot, ws, base)
        binding.oppo_chunk_prefill_attn(desc, cache, cu, q_rot, out)
        torch.cuda.synchronize()
        o = out.cpu().numpy().view(np.uint16)
        for i in range(B):
            outs[i][done[i]:done[i] + ql[i]] = o[cu[i]:cu[i + 1]]
        done += ql
    assert done.tolist() == n_tok.tolist()
    errs = []
    for i in range(B):
        q, k, v = qkv_projection_rope(xs[i], wb, np.arange(int(n_tok[i]), dtype=np.float64), Hq, Hkv, D, base)
        # the attention sees what the projection stored: bf16-rounded queries, keys and values
        rq, rk, rv = (bf16_bits_to_f64(f32_to_bf16_bits(t.astype(np.float32))) for t in (q, k, v))
        ref = full_prefill(rq, rk, rv, 1.0 / np.sqrt(D))
        errs.append(np.abs(bf16_bits_to_f64(outs[i]) - ref).ravel())
    err = np.concatenate(errs)
    assert err.max() <= 3e-2 and err.mean() <= 2e-3, f"max {err.max():.3e} mean {err.mean():.3e}"
