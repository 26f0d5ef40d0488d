"""GPU: the one-launch attention of short rows (at most four 64-key splits)
against the split kernels with their combine, which the same rows take when a
longer row shares their launch: the same bits at every split edge."""
import numpy as np
import pytest

from synth import configs, gen
from tests.gpu_common import torch_cuda
from tests.test_gpu_attention import BF16_RTOL, F32_RTOL, Case, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("H,Hkv", [(4, 4), (6, 2), (8, 2), (8, 1)])
def test_short_rows_have_the_bits_of_the_split_kernels(hd, H, Hkv):
    """Positions at and around every split edge from one key to 256, rows all
    committed, with chains inside a split and across an edge, several rows
    of a sequence; one, two and four splits a launch; float64 parity."""
    torch = torch_cuda()
    seqs = [(1, [0, 1, 3]), (60, [0, 2, 4, 9]), (63, [1, 2]), (64, [0, 1, 5]), (120, [8, 9, 20]), (127, [1, 30]),
            (128, [0]), (190, [2, 5, 40]), (250, [0, 6]), (700, [2])]
    c = Case(1, hd, H, Hkv, seqs, 4200 + hd + H)
    full, full_bits = _run(torch, c)                    # 11 splits: the split kernels
    short = [r for r in range(c.R) if c.pos[r] < 256]
    for top in (64, 128, 256):                          # one, two, four splits
        rows = [r for r in short if c.pos[r] < top]
        out, bits = _run(torch, c, rows)
        assert np.array_equal(bits, full_bits[rows]), top
        ref = c.reference(rows)
        err = np.linalg.norm(out - ref, axis=1) / np.linalg.norm(ref, axis=1)
        assert err.max() <= BF16_RTOL, err.max()
    for r in (short[0], short[5], short[-1]):           # and of a launch of their own
        assert np.array_equal(_run(torch, c, [r])[1], full_bits[[r]])


@pytest.mark.parametrize("hd,H,Hkv,nc,R", [(64, 12, 12, 200, 5), (64, 12, 12, 200, 6), (128, 4, 4, 100, 24),
                                            (128, 4, 4, 100, 25), (128, 32, 8, 150, 4), (128, 32, 8, 150, 5),
                                            (128, 64, 8, 230, 16), (128, 64, 8, 230, 17)])
def test_many_rows_of_a_prefix_have_the_bits_of_a_few(hd, H, Hkv, nc, R):
    """Eight sequences of R rows, on both sides of the row counts from which
    rows that share keys go to the split kernels: any one row of each has the
    bits it has in a launch of one row a sequence."""
    torch = torch_cuda()
    c = Case(1, hd, H, Hkv, [(nc + s, [i % 4 for i in range(R)]) for s in range(8)], 4250 + hd + R)
    _, bits = _run(torch, c)
    for i in (0, R - 1):
        rows = [s * R + i for s in range(8)]
        assert np.array_equal(_run(torch, c, rows)[1], bits[rows])


@pytest.mark.parametrize("dtype,hd", [(0, 32), (0, 64), (0, 128), (1, 32)])
@pytest.mark.parametrize("H,Hkv", [(4, 4), (6, 2), (8, 1)])
def test_one_split_rows_have_the_bits_of_the_split_kernels(dtype, hd, H, Hkv):
    """The vector kernel writes rows of at most 64 keys out at once; with a
    longer row in the launch they go through split records and the combine."""
    torch = torch_cuda()
    c = Case(dtype, hd, H, Hkv, [(1, [0, 1]), (17, [0, 3, 7]), (60, [1, 4]), (64, [0]), (90, [2])], 4300 + hd + H)
    full, full_bits = _run(torch, c)
    rows = [r for r in range(c.R) if c.pos[r] < 64]
    out, bits = _run(torch, c, rows)
    assert np.array_equal(bits, full_bits[rows])
    assert np.array_equal(_run(torch, c, rows[2:3])[1], full_bits[rows[2:3]])
    ref = c.reference(rows)
    err = np.linalg.norm(out - ref, axis=1) / np.linalg.norm(ref, axis=1)
    assert err.max() <= (BF16_RTOL if dtype == 1 else F32_RTOL), err.max()


@pytest.mark.parametrize("words", [240, 960])
def test_row_tables_of_every_upload_size(words):
    """A call's row tables of up to 240 words go to the GPU as a kernel argument,
    longer ones by a copy: a row whose chain entries are the table's last words
    has the same bits on both sides of that size and at four times it."""
    torch = torch_cuda()
    c = Case(1, 64, 4, 2, [(40, [9])], 4400)
    _, want = _run(torch, c)
    chain, coff = c.chain.copy(), c.coff.copy()
    assert np.linalg.norm(_run(torch, c)[0] - c.reference()) <= BF16_RTOL * np.linalg.norm(c.reference())
    for pad in range(words - 24, words + 2):            # a one-row table holds 8 words besides its chain
        c.chain = np.concatenate([np.full(pad, c.E - 1, np.int32), chain])
        c.coff = coff + np.int32(pad)
        assert np.array_equal(_run(torch, c)[1], want), pad


def test_short_rows_take_as_long_in_a_long_context():
    """The vector kernel's row groups follow the positions that a round's rows
    reach, not what the context could hold: the attention launches of short
    fp32 rows take the same time in either context (about twice as long with
    groups sized for the context), and the tokens are the same."""
    torch_cuda()
    from paper_2606_29223_amd import dexlib
    cfg = configs.scaled_down(configs.get("tiny-4L-d128-fp32"), vocab=512)
    cfg.update(n_heads=32, n_kv_heads=8, head_dim=64)
    w = dexlib.device_weights(cfg, gen.generate_model(cfg))
    prompts = np.random.default_rng(9).integers(0, 512, (4, 16)).astype(np.int32)
    took, toks = {}, {}
    for ctx in (64, 16384):
        dec = dexlib.Decoder(cfg, w, width_cap=8, batch=4, max_context=ctx)
        runs = []
        for _ in range(3):
            dec.prefill(prompts)
            for _ in range(4):
                dec.step()
            dec.set_timing(True)
            toks[ctx] = [dec.step().tolist() for _ in range(24)]
            ms, _, _ = dec.kernel_times()
            dec.set_timing(False)
            runs.append(ms[1] + ms[2])           # attention and combine
        dec.close()
        took[ctx] = sorted(runs)[1]
    assert toks[64] == toks[16384]
    assert took[16384] < 1.4 * took[64], took
