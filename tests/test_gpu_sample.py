"""Stochastic acceptance on the HIP path vs the oracle: every decision is an integer comparison on both sides, so the
results must agree bit for bit."""
import numpy as np
import pytest

from oracle import oracle
from paper_2507_02620_amd import synth

pytestmark = pytest.mark.gpu


def _gpu(lg, temp, token, parent, n_ver, seed, step):
    import torch
    from paper_2507_02620_amd import flowspec as fs
    T = len(token)
    res, retain, _ = fs.new_accept_buffers(T, 1)
    retain.fill_(-9)
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    fs.tree_accept_sample(d(lg), temp, d(token.astype(np.int32)), d(parent.astype(np.int32)), n_ver, seed, step, res, retain)
    out, ret = fs.accept_result_to_host(res, retain, T)
    return out.as_tuple(), ret


@pytest.mark.parametrize("seed", range(16))
def test_sampled_accept_bit_exact(seed):
    rng = np.random.default_rng(seed)
    T = int(rng.choice([1, 2, 9, 64, 65, 300, 1024]))
    vocab = int(rng.choice([2, 7, 50, 1000, 32000]))
    temp = float(rng.choice([1.0, 0.5, 1.7]))
    tree = synth.random_tree(T, int(rng.choice([3, 8, 30])), int(rng.choice([0, 2, 4])), vocab, seed, forest=bool(seed % 4 == 0))
    n_ver = int(rng.integers(0, T + 1))
    lg = (synth.random_logits(max(n_ver, 1), vocab, seed, 3) * 2).astype(np.float32)
    if seed % 2:   # make long accepted paths likely
        for r, t in synth.resolve_plants(synth.plant_path(tree, n_ver, seed, 0, 0.3, 5.0), tree, vocab):
            lg[r, t] += 6.0
    inv_temp = float(np.float32(1.0) / np.float32(temp))
    print(f"[case] T={T} n_ver={n_ver} vocab={vocab} temp={temp}", flush=True)
    for step in range(6):
        o_res, o_ret = oracle.accept_sample(lg[:max(n_ver, 1)], inv_temp, tree.token, tree.parent, n_ver, 1234 + seed, step)
        g_res, g_ret = _gpu(lg[:max(n_ver, 1)], temp, tree.token, tree.parent, n_ver, 1234 + seed, step)
        assert g_res == o_res.as_tuple(), (step, g_res, o_res.as_tuple())
        assert np.array_equal(g_ret, o_ret)


def test_sampled_accept_full_vocab_residual_and_chain():
    """Qwen-sized vocabulary with no children at the root (pure residual draw), and a 1024-node verified chain."""
    lg = synth.random_logits(1, 152064, 5, 9)
    tok, par = np.array([3], dtype=np.int32), np.array([-1], dtype=np.int32)
    for step in range(8):
        o_res, _ = oracle.accept_sample(lg, 1.0, tok, par, 1, 77, step)
        g_res, _ = _gpu(lg, 1.0, tok, par, 1, 77, step)
        assert g_res == o_res.as_tuple()
    T = 1024
    chain = np.arange(-1, T - 1, dtype=np.int32)
    token = (np.arange(T, dtype=np.int32) * 7 + 3) % 50
    lg = synth.random_logits(T, 50, 6, 9)
    lg[np.arange(T - 1), token[1:]] += 12.0
    o_res, o_ret = oracle.accept_sample(lg, 1.0, token, chain, T, 5, 0)
    g_res, g_ret = _gpu(lg, 1.0, token, chain, T, 5, 0)
    assert g_res == o_res.as_tuple() and np.array_equal(g_ret, o_ret) and o_res.n_acc > 100


def test_sampled_accept_errors():
    import torch
    from paper_2507_02620_amd import flowspec as fs
    res, retain, _ = fs.new_accept_buffers(4, 1)
    t = torch.zeros(4, dtype=torch.int32, device="cuda")
    lg = torch.zeros((1, 8), device="cuda")
    with pytest.raises(fs.FlowSpecError) as e:
        fs.tree_accept_sample(lg, 0.0, t, t, 1, 0, 0, res, retain)
    assert e.value.code == fs.FS_EINVAL
    bad = torch.tensor([-1, 2, 0, 0], dtype=torch.int32, device="cuda")
    fs.tree_accept_sample(lg, 1.0, t, bad, 1, 0, 0, res, retain)
    out, _ = fs.accept_result_to_host(res, retain, 4)
    assert out.n_acc == -1


@pytest.mark.parametrize("vocab,T,n_ver,n_child", [
    # one workgroup per row: rows on 16 bytes and not, most of the tree below one node, a star of a thousand candidates
    (4096, 40, 40, 3), (4097, 40, 33, 8), (10007, 90, 90, 60), (32000, 1024, 1024, 1000),
    # rows in chunks: the smallest vocabulary that is chunked (4 chunks) and the largest that is not, odd row lengths (scalar loads, a last
    # chunk that is no multiple of four), 4 and 3 chunks of the same rows on either side of 512 rows, 38 chunks of few rows
    (12288, 30, 5, 8), (12289, 30, 5, 8), (50257, 20, 9, 5), (32000, 600, 512, 70), (32000, 600, 513, 70), (152064, 3, 2, 2),
])
def test_sampled_accept_row_chunks_and_residual(vocab, T, n_ver, n_child):
    """Row statistics cut into chunks, candidates with duplicate tokens and tokens outside the vocabulary, residual draws behind
    rejected candidates, rows with infinities and with one weight only: bit for bit as the oracle."""
    rng = np.random.default_rng(vocab + T)
    parent = np.array([-1] + [0 if i <= n_child else int(rng.integers(1, i)) for i in range(1, T)], dtype=np.int32)
    token = rng.integers(0, vocab, T).astype(np.int32)
    token[1:T:3] = token[1]                    # duplicates among siblings
    if T > 4:
        token[4] = vocab + 5                   # never a candidate
    lg = (rng.standard_normal((n_ver, vocab)) * 2).astype(np.float32)
    lg[0, token[1]] = 2.0 + np.log(vocab)      # a heavy candidate: often accepted, otherwise struck before the residual draw
    lg[-1, ::7] = -np.inf
    if n_ver > 1:
        lg[1] = -np.inf
        lg[1, vocab - 1] = 3.0                 # all weight on the last token
    print(f"[case] vocab={vocab} T={T} n_ver={n_ver}", flush=True)
    seen = set()
    for step in range(10):
        o_res, o_ret = oracle.accept_sample(lg, 1.0, token, parent, n_ver, 99, step)
        g_res, g_ret = _gpu(lg, 1.0, token, parent, n_ver, 99, step)
        assert g_res == o_res.as_tuple(), (step, g_res, o_res.as_tuple())
        assert np.array_equal(g_ret, o_ret)
        seen.add(o_res.n_acc)
    assert len(seen) > 1                       # accepted and rejected candidates both occurred


@pytest.mark.parametrize("vocab", [1000, 32000])
def test_sampled_accept_of_logits_off_a_16_byte_boundary(vocab):
    """A row length that is a multiple of four behind a base that is not on 16 bytes: scalar loads, in one workgroup per row and in chunks."""
    import torch
    from paper_2507_02620_amd import flowspec as fs
    parent, token = np.array([-1, 0, 0], dtype=np.int32), np.array([5, 7, 9], dtype=np.int32)
    lg = synth.random_logits(3, vocab, 5, 9)
    buf = torch.zeros(3 * vocab + 1, device="cuda")
    view = buf[1:].view(3, vocab)
    view.copy_(torch.from_numpy(lg))
    assert view.data_ptr() % 16 == 4
    res, retain, _ = fs.new_accept_buffers(3, 1)
    for step in range(4):
        o_res, o_ret = oracle.accept_sample(lg, 1.0, token, parent, 3, 12, step)
        fs.tree_accept_sample(view, 1.0, torch.from_numpy(token).cuda(), torch.from_numpy(parent).cuda(), 3, 12, step, res, retain)
        g_res, g_ret = fs.accept_result_to_host(res, retain, 3)
        assert g_res.as_tuple() == o_res.as_tuple() and np.array_equal(g_ret, o_ret)


@pytest.mark.parametrize("n_child", [0, 3, 7, 8, 40])
@pytest.mark.parametrize("vocab", [1, 63, 64, 65, 255, 256, 257, 1024, 1025, 4096, 4100])
def test_sampled_accept_at_the_ends_of_the_passes(vocab, n_child):
    """Vocabularies and parts of 64 and 256 entries on either side of a pass of the residual draw, few and many rejected tokens, child
    counts that are no multiple of four; all weight on the first or the last entries in some rows."""
    rng = np.random.default_rng(vocab * 50 + n_child)
    T = n_child + 1
    parent = np.array([-1] + [0] * n_child, dtype=np.int32)
    token = rng.integers(0, vocab, T).astype(np.int32)
    print(f"[case] vocab={vocab} children={n_child}", flush=True)
    for step in range(6):
        lg = (rng.standard_normal((1, vocab)) * 2).astype(np.float32)
        if step == 1:
            lg[0, :-1] = -np.inf
        if step == 2:
            lg[0, 1:] -= 30.0
        if step >= 3:
            lg[0, token[1:]] -= 4.0            # candidates that are mostly struck
        o_res, o_ret = oracle.accept_sample(lg, 1.0, token, parent, 1, 31, step)
        g_res, g_ret = _gpu(lg, 1.0, token, parent, 1, 31, step)
        assert g_res == o_res.as_tuple(), (step, g_res, o_res.as_tuple())
        assert np.array_equal(g_ret, o_ret)


@pytest.mark.parametrize("vocab,T,n_ver,n_child", [
    # one entry on either side of the 12 chunks of 4096 from which the draw has a launch of its own, and one row on either side of
    # the 14 whose sums leave room for them
    (45056, 40, 20, 3), (45057, 40, 20, 3), (152064, 40, 13, 2), (152064, 40, 14, 2),
    # rows off 16 bytes, several blocks per chunk (12 chunks of 152064 entries), a last chunk of 1024, as many chunks as there may be and
    # more blocks than that, all of the tree below the root
    (50257, 60, 60, 1), (152064, 16, 16, 5), (300000, 100, 100, 40), (262145, 80, 70, 1), (65536, 1024, 64, 1000),
])
def test_sampled_accept_draw_in_its_own_launch(vocab, T, n_ver, n_child):
    """Residual draws spread over the chip: chunks and blocks of every length, tokens struck in them, bit for bit as the oracle."""
    test_sampled_accept_row_chunks_and_residual(vocab, T, n_ver, n_child)


@pytest.mark.parametrize("place", [0, 15, 16, 4095, 4096, 8191, 98303, 98304, 99999])
def test_sampled_accept_draw_finds_an_entry_at_the_ends(place):
    """All weight on one entry at the end of a thread's, a block's, a chunk's or the row's entries; then that entry struck, with the
    definition's default where no weight is left."""
    vocab, n_ver = 100000, 16
    parent = np.full(n_ver, 0, dtype=np.int32)
    parent[0] = -1
    for tok in ((place + 7) % vocab, place):
        token = np.full(n_ver, tok, dtype=np.int32)
        lg = np.full((n_ver, vocab), -np.inf, dtype=np.float32)
        lg[0, place] = 1.0
        lg[0, (place + 70000) % vocab] = -12.0
        for step in range(3):
            o_res, o_ret = oracle.accept_sample(lg, 1.0, token, parent, n_ver, 8, step)
            g_res, g_ret = _gpu(lg, 1.0, token, parent, n_ver, 8, step)
            assert g_res == o_res.as_tuple(), (tok, step, g_res, o_res.as_tuple())
            assert np.array_equal(g_ret, o_ret)


@pytest.mark.parametrize("vocab,rows", [(12289, 256), (12289, 257), (20001, 300), (16385, 40), (13315, 17)])
def test_sampled_accept_rows_off_16_bytes(vocab, rows):
    """Element-wise rounds of four loads and what is left behind them: chunks of 3076 to 5004 elements, a last one of a few elements less."""
    test_sampled_accept_row_chunks_and_residual(vocab, rows, rows, 5)
