"""GPU: the prompt path's kernels at the sizes where they can go wrong --
edges of every prompt-GEMM tile, rings with fewer stages than slots, packed
activations whose last k-step is not full."""
import numpy as np
import pytest

import oracle
from oracle import ar
from synth import configs, gen
from tests.gpu_common import GAP, LOGIT_RTOL, check_tokens_teacher_forced, max_rel_err, run, torch_cuda
from tests.test_gpu_gemm import _gemm, _inputs

pytestmark = pytest.mark.gpu


# (N, K, M): by the cost rule of the prompt GEMM these take, in turn, the
# 256 x 256, 256 x 128, 128 x 128 (five slots, three slots), 64 x 128, 64 x 64
# and 32 x 64 tile, each with a ragged last block in N and M and a last k-step
# only partly inside K; then one, two and five k-steps (rings that never
# fill), and more shapes between
@pytest.mark.parametrize("N,K,M", [(4112, 264, 3000), (2064, 3080, 3000), (8208, 1544, 257), (2064, 264, 3000),
                                   (8208, 264, 97), (4112, 264, 97), (784, 264, 97), (4112, 24, 300), (4112, 40, 97),
                                   (528, 136, 257), (2064, 1096, 500), (1552, 776, 500), (784, 776, 65)])
def test_prompt_gemm_tiles(N, K, M):
    """float64 parity (fp32 accumulation of bf16 products: K eps sqrt-scaled,
    the bound of the other GEMM tests), and a row's bits do not depend on the
    tile: the last 70 rows alone take a smaller one."""
    torch = torch_cuda()
    Wt, xt, W64, x64 = _inputs(torch, 1, N, K, M, 900 + N + K)
    y = _gemm(torch, 1, Wt, xt, M)
    assert np.abs(y - x64 @ W64.T).max() <= 2e-5 * np.sqrt(K) * 0.05 + 1e-6
    lo = max(0, M - 70)
    part = _gemm(torch, 1, Wt, xt[lo:].contiguous(), M - lo)
    if M - lo > 64:                              # both M-tiled (the decode kernel sums in another order)
        assert np.array_equal(part.view(np.uint32), y[lo:].view(np.uint32))


@pytest.mark.parametrize("d,F,H,Hkv,hd,P", [(80, 88, 4, 2, 32, 70), (48, 72, 2, 1, 64, 90), (144, 200, 3, 1, 128, 67),
                                             (96, 64, 5, 1, 64, 201), (64, 96, 7, 1, 128, 131)])
def test_prompt_with_unfilled_k_steps(d, F, H, Hkv, hd, P):
    """bf16 models whose widths do not fill 32-column k-steps (the packed
    activations end in zeros), with head_dim 32 (whose attention writes
    row-major and is packed afterwards) and odd numbers of query heads per kv head:
    y_0 and the next tokens follow the oracle, exit logits within 2e-2."""
    torch = torch_cuda()
    from paper_2606_29223_amd import dexlib
    cfg = configs.scaled_down(configs.get("small-12L-d768-bf16"), n_layers=2, d_model=d, d_ffn=F, vocab=512)
    cfg.update(n_heads=H, n_kv_heads=Hkv, head_dim=hd, prompt_len=P, batch=2, prompt_seeds=[7301, 7302])
    w = gen.generate_model(cfg)
    T = 4
    dec = dexlib.Decoder(cfg, dexlib.device_weights(cfg, w), explored=[2], width_cap=1, max_context=P + T)
    prompt = gen.prompts(cfg)
    tap = torch.zeros((2, cfg["vocab"]), dtype=torch.float32, device="cuda")
    dec.set_logits_tap(tap)
    toks, _ = run(dec, prompt, T)
    again = dec.prefill(prompt)
    first_logits = tap.cpu().numpy()
    dec.close()
    m = oracle.Model(cfg, gen.model_as_f64(cfg, w))
    for b in range(2):
        pl, seq = [int(t) for t in prompt[b]], [int(t) for t in toks[b]]
        assert int(again[b]) == seq[0]
        pf = m.prefill(pl)
        z0 = m.exit_logits(pf[2])
        assert max_rel_err(first_logits[b], z0) <= LOGIT_RTOL
        if seq[0] != int(np.argmax(z0)):
            assert z0.max() - z0[seq[0]] < GAP
        z = ar.depth_logits(m, pl, seq, [2], prefill=pf)
        check_tokens_teacher_forced(z[:, -1], seq)


@pytest.mark.parametrize("hd,H,Hkv,P,B", [(128, 8, 2, 2110, 8), (64, 6, 6, 1310, 16)])
def test_prompt_attention_bits_do_not_depend_on_the_batch(hd, H, Hkv, P, B):
    """The batch decides how many queries a wave of the prompt attention
    takes (one 16-query tile alone; two from 1024 workgroups on: 1056 and
    1056 here): the keys and values of the second layer, which the first
    layer's attention feeds, and y_0 are the same bits either way."""
    torch = torch_cuda()
    from paper_2606_29223_amd import dexlib
    cfg = configs.scaled_down(configs.get("small-12L-d768-bf16"), n_layers=2, d_model=256, d_ffn=256, vocab=512)
    cfg.update(n_heads=H, n_kv_heads=Hkv, head_dim=hd, prompt_len=P)
    w = dexlib.device_weights(cfg, gen.generate_model(cfg))
    prompts = np.random.default_rng(hd).integers(0, 512, (B, P)).astype(np.int32)
    got = []
    for rows in (prompts, prompts[:1], prompts[B - 1:]):
        dec = dexlib.Decoder(cfg, w, explored=[2], width_cap=1, batch=len(rows), max_context=P + 2)
        first = dec.prefill(rows)
        k, v, E = dec.kv_layout()
        n = 2 * len(rows) * Hkv * E * hd * 2
        caches = []
        for base in (k, v):
            buf = torch.empty(n, dtype=torch.uint8, device="cuda")
            assert dexlib.load().dex_debug_copy(buf.data_ptr(), base, n, dec.stream.cuda_stream) == 0
            torch.cuda.synchronize()
            caches.append(buf.view(torch.int16).view(2, len(rows), Hkv, E, hd)[1, :, :, :P].clone())
        dec.close()
        got.append((first, *caches))
    for i, b in ((1, 0), (2, B - 1)):
        assert got[i][0][0] == got[0][0][b]
        assert torch.equal(got[i][1][0], got[0][1][b]) and torch.equal(got[i][2][0], got[0][2][b])


@pytest.mark.parametrize("name", ["tiny-4L-d128-fp32", "small-12L-d768-bf16"])
def test_keys_have_the_same_bits_at_every_row_count(name):
    """Prompts of up to 64 positions run the decode GEMMs, whose variants load
    the epilogue's inputs early or late and hold one to four row blocks: the
    rotated keys and the values of the first positions are the same bits in
    all of them."""
    torch = torch_cuda()
    from paper_2606_29223_amd import dexlib
    cfg = configs.scaled_down(configs.get(name), n_layers=2, d_model=256, d_ffn=256, vocab=512)
    cfg.update(n_heads=4, n_kv_heads=2, head_dim=64)
    w = dexlib.device_weights(cfg, gen.generate_model(cfg))
    prompt = np.random.default_rng(11).integers(0, 512, (1, 64)).astype(np.int32)
    el = 2 if cfg["dtype"] == "bf16" else 4
    want = None
    for P in (64, 33, 32, 17, 16, 9, 8, 3):
        dec = dexlib.Decoder(dict(cfg, prompt_len=P), w, explored=[2], width_cap=1, batch=1, max_context=P + 2)
        dec.prefill(prompt[:, :P])
        k, v, E = dec.kv_layout()
        n = 2 * E * 64 * el                      # layer 0
        got = []
        for base in (k, v):
            buf = torch.empty(n, dtype=torch.uint8, device="cuda")
            assert dexlib.load().dex_debug_copy(buf.data_ptr(), base, n, dec.stream.cuda_stream) == 0
            torch.cuda.synchronize()
            got.append(buf.view(2, E, 64 * el)[:, :P].clone())
        dec.close()
        want = want or got
        for a, b in zip(got, want):
            assert torch.equal(a, b[:, :P]), P


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("P,B", [(46, 1), (60, 3), (200, 2), (2100, 2)])
def test_first_token_attends_with_fp32_partial_sums(hd, P, B):
    """Every row's attention is a plain mean of the values here (no query),
    each value +-1 +- 1/64, and the parts of size 1 cancel over the whole
    prompt but not within 64 keys: an output rounded to bf16 before all keys
    are in is off by about a tenth, one rounded at the end by 2^-9.  Logits
    are the final state's own components, so y_0's row shows the output."""
    torch = torch_cuda()
    from paper_2606_29223_amd import dexlib
    H, Hkv, V = 4, 2, 1024
    d, half = H * hd, V // 2
    rng = np.random.default_rng(100 * hd + P)
    x = rng.choice([-1.0, 1.0], size=(V, d))
    x[half:, d // 2:] = x[:half, d // 2:]        # token t + half: t with its first components negated
    x[half:, :d // 2] = -x[:half, :d // 2]
    wv = np.zeros((Hkv * hd, d))
    i = np.arange(Hkv * hd)
    wv[i, i % (d // 2)] = 1.0
    wv[i, d // 2 + rng.permutation(d // 2)[i % (d // 2)]] = 1.0 / 64
    alpha = 2.0 ** round(np.log2(8 * 64 * np.sqrt(P / 2.0)))
    cfg = dict(configs.get("small-12L-d768-bf16"), n_layers=1, d_model=d, n_heads=H, n_kv_heads=Hkv, head_dim=hd,
               d_ffn=16, vocab=V, rms_eps=1e-12, residual_scale=alpha, prompt_len=P, batch=B, explored=[1])
    z = lambda *s: np.zeros(s)  # noqa: E731
    one = torch.ones(d, device="cuda")
    mats = {"embed": x, "lm_head": np.eye(V, d), "layers.0.wq": z(d, d), "layers.0.wk": z(Hkv * hd, d),
            "layers.0.wv": wv, "layers.0.wo": np.eye(d), "layers.0.w_gate": z(16, d), "layers.0.w_up": z(16, d),
            "layers.0.w_down": z(d, 16)}
    w = {n: torch.as_tensor(m, dtype=torch.bfloat16, device="cuda") for n, m in mats.items()}
    w.update({"final_norm": one, "layers.0.attn_norm": one, "layers.0.ffn_norm": one})
    prompts = np.empty((B, P), np.int32)
    prompts[:, :P // 2] = rng.integers(0, half, (B, P // 2))
    prompts[:, P // 2:] = prompts[:, :P // 2] + half
    dec = dexlib.Decoder(cfg, w, width_cap=1, batch=B, max_context=P + 2)
    tap = torch.zeros((B, V), dtype=torch.float32, device="cuda")
    dec.set_logits_tap(tap)
    dec.prefill(prompts)
    got = tap.cpu().numpy()[:, :d].astype(np.float64)
    dec.close()
    for b in range(B):
        att = np.repeat((x[prompts[b]] @ wv.T).mean(0).reshape(Hkv, hd), H // Hkv, axis=0).reshape(-1)
        h = x[prompts[b, -1]] + alpha * att
        r = 1.0 / np.sqrt(np.mean(h * h))
        # att and the head's input are each rounded to bf16 (2^-9 of the value), which moves the
        # scale r by as much at most; a tenth for the fp32 operations beside them
        bound = 1.1 * 2.0 ** -9 * r * (alpha * np.abs(att) + 2 * np.abs(h)) + 1e-6
        assert (np.abs(got[b] - r * h) <= bound).all(), (np.abs(got[b] - r * h) / bound).max()


def _pinned_bytes(torch):
    """GPU driver mappings of this process beyond the device memory in use."""
    spans = [line.split()[0].split("-") for line in open("/proc/self/maps") if "/dev/dri/renderD" in line]
    free, total = torch.cuda.mem_get_info()
    return sum(int(hi, 16) - int(lo, 16) for lo, hi in spans) - (total - free)


def test_prompt_keeps_no_host_memory_that_grows_with_it():
    """Row tables of a million prompt rows (12 MB) are gone after the call: a
    context keeps 1 MiB of pinned tables at most."""
    torch = torch_cuda()
    from paper_2606_29223_amd import dexlib
    B, P = 64, 16384
    cfg = configs.scaled_down(configs.get("small-12L-d768-bf16"), n_layers=1, d_model=64, d_ffn=64, vocab=512)
    cfg.update(n_heads=1, n_kv_heads=1, head_dim=64, prompt_len=P)
    w = dexlib.device_weights(cfg, gen.generate_model(cfg))
    dec = dexlib.Decoder(cfg, w, explored=[1], width_cap=1, batch=B, max_context=P + 2)
    long = np.random.default_rng(4).integers(0, 512, (B, P)).astype(np.int32)
    short = np.ascontiguousarray(long[:, :64])
    first = dec.prefill(short)
    before = _pinned_bytes(torch)
    dec.prefill(long)
    assert np.array_equal(dec.prefill(short), first)
    assert _pinned_bytes(torch) - before < 4 << 20
    dec.close()


def test_prompt_after_one_that_found_no_memory():
    """A prompt whose scratch (1.2 GB) does not fit fails with DEX_E_NOMEM and
    leaves the context as it was: the next one, with memory back, succeeds."""
    torch = torch_cuda()
    from paper_2606_29223_amd import dexlib
    P = 8192
    cfg = configs.scaled_down(configs.get("small-12L-d768-bf16"), n_layers=1, d_model=128, d_ffn=65536, vocab=512)
    cfg.update(n_heads=2, n_kv_heads=1, head_dim=64, prompt_len=P)
    w = dexlib.device_weights(cfg, gen.generate_model(cfg))
    prompt = np.random.default_rng(6).integers(0, 512, (1, P)).astype(np.int32)
    dec = dexlib.Decoder(cfg, w, explored=[1], width_cap=1, batch=1, max_context=P + 2)
    torch.cuda.empty_cache()
    held = torch.empty(torch.cuda.mem_get_info()[0] - (64 << 20), dtype=torch.uint8, device="cuda")
    try:
        with pytest.raises(dexlib.DexError) as e:
            dec.prefill(prompt)
        assert e.value.status == dexlib.DEX_E_NOMEM
    finally:
        del held
        torch.cuda.empty_cache()
    first = dec.prefill(prompt)
    dec.step()
    dec.close()
    fresh = dexlib.Decoder(cfg, w, explored=[1], width_cap=1, batch=1, max_context=P + 2)
    assert np.array_equal(fresh.prefill(prompt), first)
    fresh.close()
