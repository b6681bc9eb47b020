"""Matrices of 4 GiB and more: the kernels that address their operands with 32-bit offsets do not take them, the few-row kernels do."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

GIB4 = 1 << 32


def _normed(x, eps):
    x = x.float()
    return x * (x.square().mean(dim=1, keepdim=True) + eps).rsqrt()


def _rel(got, ref):
    return float((got.float() - ref).abs().max() / ref.abs().max())


def test_dense_projection_and_head_of_4_gib():
    """QKV and LM head (510 feature blocks, a count that the few-row kernel takes at 17 rows) of a stage with d_model 33024: the V rows
    in the cache and the logits against float32 products, the hidden states of 17 rows against those of its first 16 rows alone."""
    import torch
    from paper_2507_02620_amd import flowspec as fs
    d, h, hd, f, vocab, rows = 33024, 171, 128, 32, 65280, 17
    assert 2 * 3 * h * hd * d >= GIB4 and 2 * vocab * d >= GIB4
    print("[case] dense 4 GiB", flush=True)
    g = torch.Generator(device="cuda").manual_seed(3)
    mat = lambda n, k: torch.empty((n, k), dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.01, generator=g)  # noqa: E731
    one = torch.ones(d, dtype=torch.bfloat16, device="cuda")
    lw = {"rms_attn": one, "rms_ffn": one, "wq": mat(h * hd, d), "wk": mat(h * hd, d), "wv": mat(h * hd, d), "wo": mat(d, h * hd),
          "w_gate": mat(f, d), "w_up": mat(f, d), "w_down": mat(d, f)}
    lm = mat(vocab, d)
    st = fs.Stage(n_layers=1, d_model=d, n_q_heads=h, n_kv_heads=h, head_dim=hd, d_ffn=f, vocab=vocab, dtype=fs.FS_BF16, rms_eps=1e-5, rope_theta=1e4,
                  kv_capacity=32, max_tree=32, max_seg=32, layers=[lw], final_norm=one, lm_head=lm)
    kv = st.new_kv_cache()
    hid = torch.empty((rows, d), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    par = np.array([-1] + [i // 2 for i in range(rows - 1)], dtype=np.int32)
    x = _normed(hid, 1e-5)
    out16 = st.tree_verify_stage(kv, 0, 0, hid[:16].contiguous(), 0, par[:16]).clone()
    kv.zero_()
    out = st.tree_verify_stage(kv, 0, 0, hid, 0, par)
    v = torch.cat([x @ lw["wv"][i:i + 2048].float().t() for i in range(0, h * hd, 2048)], dim=1)
    logits, amax = st.tree_logits(hid)
    ref = torch.cat([x @ lm[i:i + 4096].float().t() for i in range(0, vocab, 4096)], dim=1)
    errs = _rel(kv[0, 1, :, :rows].transpose(0, 1).reshape(rows, -1), v), _rel(out[:16], out16.float()), _rel(logits, ref)
    print("  V rows %.2e, hidden %.2e, logits %.2e" % errs, flush=True)
    assert max(errs) < 2e-2
    assert torch.equal(amax.long(), logits.argmax(dim=1))


def test_4bit_head_of_4_gib():
    """33 rows, which the many-row 4-bit kernel would take, times 4 GiB of codes."""
    import torch
    from paper_2507_02620_amd import flowspec as fs
    d, hd, f, vocab, rows = 32768, 128, 128, 262144, 33
    assert vocab * d // 2 >= GIB4
    print("[case] 4-bit 4 GiB", flush=True)
    g = torch.Generator(device="cuda").manual_seed(4)
    lw = {"rms_attn": torch.ones(d, dtype=torch.bfloat16, device="cuda"), "rms_ffn": torch.ones(d, dtype=torch.bfloat16, device="cuda")}
    codes = lambda n, k: torch.randint(0, 256, (n, k // 2), dtype=torch.uint8, device="cuda", generator=g)  # noqa: E731
    scales = lambda n, k: (torch.rand((n, k // 128), device="cuda", generator=g) * 4e-3 + 1e-3).to(torch.bfloat16)  # noqa: E731
    for name, sname, n, k in (("wq", "sq", hd, d), ("wk", "sk", hd, d), ("wv", "sv", hd, d), ("wo", "so", d, hd), ("w_gate", "s_gate", f, d),
                              ("w_up", "s_up", f, d), ("w_down", "s_down", d, f)):
        lw[name], lw[sname] = codes(n, k), scales(n, k)
    lm, lms = codes(vocab, d), scales(vocab, d)
    st = fs.Stage(n_layers=1, d_model=d, n_q_heads=1, n_kv_heads=1, head_dim=hd, d_ffn=f, vocab=vocab, dtype=fs.FS_BF16, rms_eps=1e-5, rope_theta=1e4,
                  kv_capacity=64, max_tree=64, max_seg=64, layers=[lw], final_norm=lw["rms_attn"], lm_head=lm, lm_head_scale=lms,
                  weight_format=fs.FS_WFMT_INT4_G128)
    hid = torch.empty((rows, d), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    logits, amax = st.tree_logits(hid)
    x, worst, top = _normed(hid, 1e-5), 0.0, 0.0
    for i in range(0, vocab, 8192):
        c = lm[i:i + 8192]
        w = (torch.stack((c & 15, c >> 4), dim=2).view(8192, -1, 128).float() - 8.0) * lms[i:i + 8192].float()[:, :, None]
        ref = x @ w.view(8192, d).t()
        worst, top = max(worst, float((logits[:, i:i + 8192] - ref).abs().max())), max(top, float(ref.abs().max()))
    print("  logits %.2e" % (worst / top), flush=True)
    assert worst < 2e-2 * top
    assert torch.equal(amax.long(), logits.argmax(dim=1))
