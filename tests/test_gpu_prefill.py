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
    activations end in zeros), with head_dim 32 (whose attention is the split
    kernel with its combine) and odd numbers of query heads per kv head:
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


def _second_layer(torch, hd, H, Hkv, prompts, cfg, w):
    """y_0 and the second layer's keys and values (bf16 bits), which the first
    layer's attention feeds."""
    from paper_2606_29223_amd import dexlib
    B, P = prompts.shape
    dec = dexlib.Decoder(cfg, w, explored=[2], width_cap=1, batch=B, max_context=P + 2)
    first = dec.prefill(prompts)
    k, v, E = dec.kv_layout()
    n = 2 * B * Hkv * E * hd * 2
    caches = []
    for base in (k, v):
        buf = torch.empty(n, dtype=torch.uint8, device="cuda")
        assert dexlib.load().dex_debug_copy(buf.data_ptr(), base, n, dec.stream.cuda_stream) == 0
        torch.cuda.synchronize()
        caches.append(buf.view(torch.int16).view(2, B, Hkv, E, hd)[1, :, :, :P].clone())
    dec.close()
    return first, caches[0], caches[1]


def _attention_workgroups(H, Hkv, B, P):
    """Workgroups of a prompt's largest attention launch, two query tiles a
    wave: a launch takes whole sequences, about 8192 rows of them."""
    parts = -(-B // max(1, 8192 // P))
    span = 32 * max(1, 4 // (H // Hkv))
    return -(-P // span) * Hkv * -(-B // parts)


def _two_layer_model(hd, H, Hkv, P, d=256, F=256):
    from paper_2606_29223_amd import dexlib
    cfg = configs.scaled_down(configs.get("small-12L-d768-bf16"), n_layers=2, d_model=d, d_ffn=F, vocab=512)
    cfg.update(n_heads=H, n_kv_heads=Hkv, head_dim=hd, prompt_len=P)
    return cfg, dexlib.device_weights(cfg, gen.generate_model(cfg))


def _second_layer_f64(torch, cfg, w, tokens):
    """The second layer's keys and values [Hkv][P][hd] of one prompt in float64."""
    d, H, Hkv, hd = cfg["d_model"], cfg["n_heads"], cfg["n_kv_heads"], cfg["head_dim"]
    P = len(tokens)
    W = {n: (t.view(torch.bfloat16) if t.dtype == torch.int16 else t).double() for n, t in w.items()}
    ang = torch.arange(P, device="cuda").double()[:, None] * cfg["rope_theta"] ** (
        -2.0 * torch.arange(hd // 2, device="cuda").double() / hd)
    c, s = torch.cos(ang)[:, None], torch.sin(ang)[:, None]

    def norm(h, g):
        return h * torch.rsqrt(h.pow(2).mean(-1, keepdim=True) + cfg["rms_eps"]) * g

    def rope(y):
        y = y.view(P, -1, hd)
        a, b = y[..., :hd // 2], y[..., hd // 2:]
        return torch.cat((a * c - b * s, b * c + a * s), -1)

    h = W["embed"][torch.as_tensor(tokens, device="cuda", dtype=torch.long)]
    for l in range(2):
        p = f"layers.{l}."
        x = norm(h, W[p + "attn_norm"])
        k, v = rope(x @ W[p + "wk"].T), (x @ W[p + "wv"].T).view(P, Hkv, hd)
        if l == 1:
            return k.transpose(0, 1), v.transpose(0, 1)
        q = rope(x @ W[p + "wq"].T)
        mask = torch.ones(P, P, device="cuda", dtype=torch.bool).triu(1)
        att = torch.empty_like(q)
        for i in range(H):
            sc = (q[:, i] @ k[:, i // (H // Hkv)].T / hd ** 0.5).masked_fill(mask, -float("inf"))
            att[:, i] = torch.softmax(sc, -1) @ v[:, i // (H // Hkv)]
        alpha = cfg["residual_scale"] / cfg["n_layers"]
        h = h + alpha * (att.reshape(P, -1) @ W[p + "wo"].T)
        x = norm(h, W[p + "ffn_norm"])
        h = h + alpha * ((torch.nn.functional.silu(x @ W[p + "w_gate"].T) * (x @ W[p + "w_up"].T)) @ W[p + "w_down"].T)


@pytest.mark.parametrize("hd,H,Hkv,P,B", [(128, 32, 8, 1010, 8), (64, 32, 8, 1010, 8), (64, 24, 12, 1000, 8)])
def test_prompt_attention_of_one_and_two_query_tiles(hd, H, Hkv, P, B):
    """The batch decides how many queries a wave of the prompt attention takes
    (one 16-query tile; two once the launch has 1024 workgroups): the keys and
    values of the second layer and y_0 are the same bits either way, and
    those of the two-tile launch follow float64 (bf16 inputs, weights and
    caches: 2^-9 each over a layer, about 3e-3 of the norm)."""
    torch = torch_cuda()
    assert _attention_workgroups(H, Hkv, B, P) >= 1024 > _attention_workgroups(H, Hkv, 1, P)
    cfg, w = _two_layer_model(hd, H, Hkv, P)
    prompts = np.random.default_rng(hd + H).integers(0, 512, (B, P)).astype(np.int32)
    both = _second_layer(torch, hd, H, Hkv, prompts, cfg, w)
    for b in (0, B - 1):
        first, k, v = _second_layer(torch, hd, H, Hkv, prompts[b:b + 1], cfg, w)
        assert first[0] == both[0][b]
        assert torch.equal(k[0], both[1][b]) and torch.equal(v[0], both[2][b])
    for got, ref in zip(both[1:], _second_layer_f64(torch, cfg, w, prompts[B - 1])):
        d = got[B - 1].view(torch.bfloat16).double() - ref
        assert float(d.norm() / ref.norm()) <= 1e-2
        rows = d.pow(2).sum((0, 2)).sqrt() / ref.pow(2).sum((0, 2)).sqrt()
        assert float(rows.max()) <= 2e-2, int(rows.argmax())


def test_prompt_layer_on_the_largest_tile():
    """A 2048-wide layer at 8 x 775 rows: by the cost rule of the prompt GEMM all
    four projections take the 256 x 256 tile (QKV with RoPE and the cache write,
    O and down with the residual, gate/up with SwiGLU), one sequence alone
    smaller ones.  The second layer's keys and values, which pass through
    every one of them, are the same bits and follow float64."""
    torch = torch_cuda()
    hd, H, Hkv, P, B = 128, 16, 8, 775, 8
    cfg, w = _two_layer_model(hd, H, Hkv, P, 2048, 4096)
    prompts = np.random.default_rng(12).integers(0, 512, (B, P)).astype(np.int32)
    both = _second_layer(torch, hd, H, Hkv, prompts, cfg, w)
    first, k, v = _second_layer(torch, hd, H, Hkv, prompts[B - 1:], cfg, w)
    assert first[0] == both[0][B - 1]
    assert torch.equal(k[0], both[1][B - 1]) and torch.equal(v[0], both[2][B - 1])
    for got, ref in zip(both[1:], _second_layer_f64(torch, cfg, w, prompts[B - 1])):
        assert float((got[B - 1].view(torch.bfloat16).double() - ref).norm() / ref.norm()) <= 1e-2


@pytest.mark.parametrize("name,P,B", [("tiny-4L-d128-fp32", 1500, 7), ("hd32-bf16", 1500, 7), ("tiny-4L-d128-fp32", 9001, 1),
                                      ("hd32-bf16", 300, 64)])
def test_split_kernel_prompts_in_parts(name, P, B):
    """Prompts whose attention is the vector split kernel (fp32; bf16 with
    head_dim 32), of more than 8192 rows: parts of whole sequences, each with
    its own row groups and chunks (4 + 3 sequences, one long one, 22 + 22 + 20).
    Every sequence has the caches and y_0 of itself alone, and the first
    follows float64."""
    torch = torch_cuda()
    from paper_2606_29223_amd import dexlib
    if name == "hd32-bf16":
        cfg = configs.scaled_down(configs.get("small-12L-d768-bf16"), n_layers=2, d_model=128, d_ffn=256, vocab=512)
        cfg.update(n_heads=4, n_kv_heads=2, head_dim=32)
    else:
        cfg = configs.scaled_down(configs.get(name), n_layers=2)
    bf16, Hkv, hd = cfg["dtype"] == "bf16", cfg["n_kv_heads"], cfg["head_dim"]
    cfg["prompt_len"] = P
    w = dexlib.device_weights(cfg, gen.generate_model(cfg))
    prompts = np.random.default_rng(P + B).integers(0, cfg["vocab"], (B, P)).astype(np.int32)

    def prefill(rows):
        dec = dexlib.Decoder(cfg, w, explored=[2], width_cap=1, batch=len(rows), max_context=P + 2)
        first = dec.prefill(rows)
        kp, vp, E = dec.kv_layout()
        n = 2 * len(rows) * Hkv * E * hd * (2 if bf16 else 4)
        out = []
        for base in (kp, vp):
            buf = torch.empty(n, dtype=torch.uint8, device="cuda")
            assert dexlib.load().dex_debug_copy(buf.data_ptr(), base, n, dec.stream.cuda_stream) == 0
            torch.cuda.synchronize()
            t = buf.view(torch.int16 if bf16 else torch.int32).view(2, len(rows), Hkv, E, hd)
            out.append(t[1, :, :, :P].clone())
        dec.close()
        return first, out[0], out[1]

    both = prefill(prompts)
    for b in sorted({0, B // 2, B - 1}):
        first, k, v = prefill(prompts[b:b + 1])
        assert first[0] == both[0][b]
        assert torch.equal(k[0], both[1][b]) and torch.equal(v[0], both[2][b])
    for got, ref in zip(both[1:], _second_layer_f64(torch, cfg, w, prompts[0])):
        d = got[0].view(torch.bfloat16 if bf16 else torch.float32).double() - ref
        assert float(d.norm() / ref.norm()) <= (1e-2 if bf16 else 2e-6)


@pytest.mark.parametrize("hd,H,Hkv,P,B", [(128, 8, 2, 2110, 8), (64, 6, 6, 1310, 16)])
def test_prompt_attention_bits_do_not_depend_on_the_batch(hd, H, Hkv, P, B):
    """Batches of more than 8192 rows run in parts of whole sequences (3 + 3 + 2
    and 6 + 6 + 4 here): the keys and values of the second layer, which the first
    layer's attention feeds, and y_0 have the bits of each sequence alone."""
    torch = torch_cuda()
    cfg, w = _two_layer_model(hd, H, Hkv, P)
    prompts = np.random.default_rng(hd).integers(0, 512, (B, P)).astype(np.int32)
    got = [_second_layer(torch, hd, H, Hkv, rows, cfg, w) for rows in (prompts, prompts[:1], prompts[B - 1:])]
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
