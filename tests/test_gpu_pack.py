"""sfl_pack_twell on the GPU is bit-exact against the oracle's extractor and classifier
on the same float32 pre-activations (Alg. 1 + the hybrid classification of Sec. 3.4)."""
import numpy as np
import pytest
import torch

from oracle import twell
from tests.gpu_util import assert_twell_equal, dev, host_bits, twell_views

pytestmark = pytest.mark.gpu

b = pytest.importorskip("paper_2603_23198_amd.binding")
from tests.test_gpu_packed32 import assert_words_equal, got_words  # noqa: E402


def special_z(T, f, seed, density=0.05):
    r = np.random.default_rng(seed)
    Z = r.standard_normal((T, f)).astype(np.float32)
    if Z.size == 0:
        return Z
    Z -= np.float32(np.quantile(Z, 1 - density))
    n = T * f
    pick = r.choice(n, size=min(n, 200), replace=False)
    specials = np.array([0.0, -0.0, np.nan, np.inf, -np.inf, 1e-45, -1e-45, 1.1754942e-38,
                         3.4028235e38, 1.0 + 2 ** -8, 1.0 + 3 * 2 ** -8], dtype=np.float32)
    Z.reshape(-1)[pick] = specials[np.arange(len(pick)) % len(specials)]
    return Z


CASES = [
    # T, f, T_n, S, K, cap, dtype
    (37, 300, 256, 32, 8, 0, "bf16"),
    (64, 1024, 256, 32, 32, 0, "f32"),
    (129, 777, 64, 4, 12, 0, "bf16"),
    (50, 97, 3, 2, 5, 0, "f32"),
    (33, 12, 5, 1, 2, 0, "bf16"),
    (300, 4096, 128, 8, 100, 7, "bf16"),     # capacity below the number of overflow rows
    (1, 65535, 256, 32, 2000, 0, "bf16"),    # largest index
    (0, 256, 256, 32, 8, 0, "bf16"),         # empty
    # up to 256 rows with f a multiple of 64: one workgroup per row packs and classifies
    (200, 2048, 64, 16, 40, 0, "bf16"),
    (256, 4096, 128, 8, 100, 7, "bf16"),     # capacity below the number of overflow rows
    (3, 1984, 256, 32, 64, 0, "bf16"),       # partial last tile
    (17, 320, 128, 128, 500, 0, "f32"),      # every column of a tile kept
    (2, 24576, 256, 32, 400, 0, "bf16"),     # a row of 96 KB of fp32 in LDS
    # above 256 rows with f at most 768: pack and classification apart
    (257, 4, 64, 4, 2, 0, "bf16"),
    (300, 260, 256, 16, 14, 0, "bf16"),      # partial last tile
    (8300, 132, 64, 12, 12, 0, "f32"),
    (300, 768, 256, 16, 40, 0, "bf16"),
    # f above that and a multiple of 4: four waves per row pack and classify
    (700, 1284, 128, 16, 60, 9, "f32"),      # partial last step, capacity below the overflow rows
    (513, 1024, 64, 8, 0, 0, "bf16"),        # every active row is a dense-backup row
    (300, 772, 256, 16, 40, 0, "bf16"),      # the fourth wave with one lane of columns
    (300, 8192, 256, 32, 1011, 0, "bf16"),   # the widest ELL rows the waves' LDS holds
    (300, 8192, 256, 32, 1012, 0, "bf16"),   # wider: pack and classification apart
    (300, 8192, 128, 32, 722, 0, "f32"),     # the widest in float32
    (301, 4096, 256, 256, 40, 0, "bf16"),    # quarters of a row on both sides of K entries
    (1501, 1284, 256, 24, 80, 0, "bf16"),    # more rows than 256 blocks take at once
    (4097, 772, 64, 16, 50, 0, "f32"),       # than 512 blocks, the last block with one row
]


@pytest.mark.parametrize("T,f,Tn,S,K,cap,dt", CASES)
def test_pack_bit_exact(T, f, Tn, S, K, cap, dt):
    Z = special_z(T, f, seed=T * 7 + f)
    if T > 3:
        Z[1] = 1.0        # all-active row: tile and row overflow
        Z[2] = -1.0       # all-inactive row
    cfg = b.make_cfg(tile_cols=Tn, tile_slots=S, ell_width=K, ovf_capacity=cap)
    bufs = b.alloc_twell(T, f, dt, cfg)
    stats = b.alloc_stats()
    b.sfl_pack_twell(dev(Z), dt, cfg, bufs, stats)
    torch.cuda.synchronize()
    tw = twell.extract_twell(Z, Tn, S, dt)
    hy = twell.classify(tw, K)
    got = twell_views(bufs, T, f, cfg)
    assert_twell_equal(got, tw, hy)
    n_ovf = len(hy.ovf_rows)
    assert got["n_ovf"] == n_ovf
    capv = cap if cap else T
    np.testing.assert_array_equal(got["ovf_rows"][:min(n_ovf, capv)], hy.ovf_rows[:capv])
    st = b.read_stats(stats)
    assert st["total_nnz"] == int(tw.cnt.sum())
    assert st["n_ovf_rows"] == n_ovf
    assert st["n_tile_ovf"] == hy.n_tile_ovf
    assert st["capacity_exceeded"] == int(n_ovf > capv)


@pytest.mark.parametrize("Tn,S,K,dt,packed", [(256, 32, 100, "bf16", False), (256, 256, 130, "bf16", False),
                                              (128, 128, 100, "f32", False), (64, 8, 722, "f32", False),
                                              (256, 31, 100, "bf16", True), (128, 31, 130, "bf16", True),
                                              (64, 31, 1011, "bf16", True)])
def test_rows_turn_dense_anywhere(Tn, S, K, dt, packed):
    """Four waves per row, three groups of steps per wave (f = 13000): rows that exceed the ELL
    width or a tile's slots in the first, a middle or the last step of a quarter, in one quarter
    only, throughout or not at all: the slabs (planes or packed words), counts, flags, ELL rows
    and statistics are the oracle's bit for bit."""
    T, f, quarter = 301, 13000, 3328
    r = np.random.default_rng(Tn + S + K)
    Z = -np.abs(r.standard_normal((T, f)).astype(np.float32)) - np.float32(0.1)
    on = np.zeros((T, f), dtype=bool)
    on[0::10] = r.random((len(on[0::10]), f)) < 0.0005
    on[1::10] = r.random((len(on[1::10]), f)) < 0.7 * K / f
    on[2::10] = True
    for q in range(4):
        on[4::10, q * quarter + 3072:(q + 1) * quarter] = True   # the last step of every quarter
        on[5::10, q * quarter + 1700:q * quarter + 1900] = True  # in the second group
        on[6::10, q * quarter:q * quarter + 9] = True            # one tile, in the first step
    on[7::10] = r.random((len(on[7::10]), f)) < 0.1
    on[8::10, quarter:2 * quarter] = True                        # one quarter only
    on[9::10, -1::-20] = True
    Z[on] *= -1
    layout = b.SFL_TWELL_PACKED32 if packed else 0
    cfg = b.make_cfg(tile_cols=Tn, tile_slots=S, ell_width=K, layout=layout)
    bufs, stats = b.alloc_twell(T, f, dt, cfg), b.alloc_stats()
    b.sfl_pack_twell(dev(Z), dt, cfg, bufs, stats)
    torch.cuda.synchronize()
    tw = twell.extract_twell(Z, Tn, S, dt)
    hy = twell.classify(tw, K)
    if packed:
        assert_words_equal(got_words(bufs, T, f, Tn), twell.pack32(tw))
        for name in ("row_nnz", "row_ovf"):
            np.testing.assert_array_equal(host_bits(bufs[name])[:T], {"row_nnz": hy.row_nnz, "row_ovf": hy.is_ovf}[name])
        for name in ("ell_idx", "ell_val"):
            got, want = host_bits(bufs[name])[:T * K].reshape(T, K), getattr(hy, name)
            used = (np.arange(K) < hy.row_nnz[:, None]) & ~hy.is_ovf[:, None]
            np.testing.assert_array_equal(got[used], want[:, :K][used])
    else:
        assert_twell_equal(twell_views(bufs, T, f, cfg), tw, hy)
    st = b.read_stats(stats)
    assert 0 < len(hy.ovf_rows) < T and st["n_ovf_rows"] == len(hy.ovf_rows)
    assert st["total_nnz"] == int(tw.cnt.sum()) and st["n_tile_ovf"] == hy.n_tile_ovf
    kept = twell.stored_to_f64(hy.ell_val, dt).sum()
    assert abs(st["l1_sum"] - kept) <= 1e-5 * kept


def test_pack_is_deterministic():
    Z = special_z(512, 4096, seed=5, density=0.02)
    cfg = b.make_cfg(tile_cols=256, tile_slots=32, ell_width=128)
    outs = []
    for _ in range(3):
        bufs = b.alloc_twell(512, 4096, "bf16", cfg)
        for v in bufs.values():
            if v is not None:
                v.zero_()
        b.sfl_pack_twell(dev(Z), "bf16", cfg, bufs)
        torch.cuda.synchronize()
        outs.append({k: v.cpu().clone() for k, v in bufs.items() if v is not None})
    for o in outs[1:]:
        for k in o:
            assert torch.equal(o[k].view(torch.uint8), outs[0][k].view(torch.uint8)), k
