"""GPU parity of the pipeline ends (token embedding; final norm + vocabulary projection + greedy
selection) against oracle/ends_oracle.py, through the C ABI.

Index work (the lookup, the selection on given logits) must be bit-exact.  Logits are fp32 with
fp32 accumulation over bf16 operands: row-normalised tolerance 1e-2 against the fp64 oracle.  The
selected token is a floating-point decision: where the oracle's two best logits are further apart
than the logits tolerance the GPU must pick the same token, otherwise it must pick a token whose
oracle logit is within that tolerance of the best (any of the near-ties is a valid answer)."""
import numpy as np
import pytest
import torch

from harness import workload as W
from oracle import ends_oracle as E
from oracle import stage_oracle as O
from paper_2506_10470_amd import tdp
from stage_helpers import Stage, f64, i32, oracle_layers, oracle_shape, row_rel_err

pytestmark = pytest.mark.gpu
LOGIT_TOL = 1e-2


class Ends:
    def __init__(self, sh, vocab, max_tokens):
        self.sh, self.vocab = sh, vocab
        self.h = tdp.tdp_ends_create(tdp.EndsConfig(vocab, sh.d_model, sh.rms_eps, max_tokens))
        self.table = W.ends_weight(sh, "embedding", vocab, device="cuda")
        self.head = W.ends_weight(sh, "lm_head", vocab, device="cuda")
        self.gain = W.ends_weight(sh, "final_norm", vocab, device="cuda", dtype=torch.float32)
        tdp.tdp_ends_set_weight(self.h, tdp.E_EMBEDDING, self.table, tdp.BF16, tdp.DEVICE, vocab, sh.d_model)
        tdp.tdp_ends_set_weight(self.h, tdp.E_LM_HEAD, self.head, tdp.BF16, tdp.DEVICE, sh.d_model, vocab)
        tdp.tdp_ends_set_weight(self.h, tdp.E_FINAL_NORM, self.gain, tdp.F32, tdp.DEVICE, sh.d_model, 1)

    def close(self):
        tdp.tdp_ends_destroy(self.h)

    def __enter__(self):
        return self

    def __exit__(self, *a):
        self.close()


def check_tokens(got_tokens, ref_logits):
    scale = np.max(np.abs(ref_logits), axis=1)
    best = E.greedy_tokens(ref_logits)
    exact = 0
    for r, tok in enumerate(got_tokens):
        row = ref_logits[r]
        srt = np.sort(row)
        gap = srt[-1] - srt[-2]
        if gap > 2 * LOGIT_TOL * scale[r]:
            assert tok == best[r], (r, tok, best[r])
            exact += 1
        else:
            assert row[best[r]] - row[tok] <= 2 * LOGIT_TOL * scale[r], (r, tok, best[r])
    return exact


def test_embedding_lookup_is_bit_exact():
    sh = W.SHAPES["tiny"]
    vocab = 1000
    with Ends(sh, vocab, 64) as e:
        ids = W.token_ids(vocab, 300, 1)
        ids[:4] = [0, vocab - 1, 0, vocab - 1]
        out = torch.full((300, sh.d_model), float("nan"), dtype=torch.bfloat16, device="cuda")
        tdp.tdp_embed_tokens(e.h, i32(ids), 300, out)
        torch.cuda.synchronize()
        ref = E.embed(ids, f64(e.table))
        assert np.array_equal(f64(out), ref)
        tdp.tdp_embed_tokens(e.h, i32(ids), 0, out)          # empty batch is a no-op


def test_embedding_host_fp32_source_and_out_of_range_ids():
    sh = W.SHAPES["tiny"]
    vocab = 64
    h = tdp.tdp_ends_create(tdp.EndsConfig(vocab, sh.d_model, 1e-5, 8))
    table = W.ends_weight(sh, "embedding", vocab, dtype=torch.float32).contiguous()
    tdp.tdp_ends_set_weight(h, tdp.E_EMBEDDING, table.numpy(), tdp.F32, tdp.HOST, vocab, sh.d_model)
    ids = np.array([3, -5, vocab + 7, 63], dtype=np.int32)
    out = torch.empty((4, sh.d_model), dtype=torch.bfloat16, device="cuda")
    tdp.tdp_embed_tokens(h, i32(ids), 4, out)
    torch.cuda.synchronize()
    ref = f64(table.to(torch.bfloat16))
    assert np.array_equal(f64(out), ref[[3, 0, vocab - 1, 63]])       # bad ids are clamped, never read wild
    tdp.tdp_ends_destroy(h)


def test_argmax_is_bit_exact_with_planted_ties():
    rng = np.random.default_rng(5)
    M, n, ld = 37, 1003, 1010
    logits = rng.integers(-3, 4, size=(M, ld)).astype(np.float32)       # few distinct values: ties everywhere
    logits[0, :n] = 1.0                                                  # all equal -> 0
    logits[1, :n] = -np.inf
    logits[1, 700] = -5.0
    logits[2, :n] = 2.0
    logits[2, n - 1] = 9.0                                               # maximum in the last column
    logits[3, n:] = 100.0                                                # padding beyond n must be ignored
    logits[4, :n] = np.nan                                               # a row of NaNs gives 0
    logits[5, 10] = np.nan
    d = torch.from_numpy(logits).cuda()
    out = torch.full((M,), -1, dtype=torch.int32, device="cuda")
    tdp.tdp_argmax_rows(d, M, n, ld, out)
    torch.cuda.synchronize()
    ref = E.greedy_tokens(np.where(np.isnan(logits[:, :n]), -np.inf, logits[:, :n]).astype(np.float64))
    ref[4] = 0
    assert np.array_equal(out.cpu().numpy(), ref)
    big = rng.standard_normal((5, 32000)).astype(np.float32)
    big[2, 31999] = 50.0
    big[3, 123] = big[3, 20000] = 40.0
    out2 = torch.empty(5, dtype=torch.int32, device="cuda")
    tdp.tdp_argmax_rows(torch.from_numpy(big).cuda(), 5, 32000, 32000, out2)
    assert np.array_equal(out2.cpu().numpy(), E.greedy_tokens(big.astype(np.float64)))


@pytest.mark.parametrize("M,vocab,use_index", [(5, 1000, False), (40, 32000, True), (257, 4096, False), (1, 260, True)])
def test_lm_head_logits_and_tokens(M, vocab, use_index):
    sh = W.SHAPES["tiny"]
    with Ends(sh, vocab, max(M, 2)) as e:
        n_rows = M * 3 if use_index else M
        x = W.hidden_states(sh, n_rows, 7, device="cuda")
        idx = (np.arange(M) * 3 + 2).astype(np.int32) if use_index else None
        logits = torch.full((M, vocab), float("nan"), dtype=torch.float32, device="cuda")
        toks = torch.full((M,), -1, dtype=torch.int32, device="cuda")
        tdp.tdp_lm_head(e.h, x, n_rows, i32(idx) if use_index else None, M, logits, toks)
        toks2 = torch.full((M,), -1, dtype=torch.int32, device="cuda")
        tdp.tdp_lm_head(e.h, x, n_rows, i32(idx) if use_index else None, M, None, toks2)   # internal logits
        torch.cuda.synchronize()
        xs = f64(x)[idx] if use_index else f64(x)
        ref = E.final_logits(xs, f64(e.gain), f64(e.head), sh.rms_eps)
        assert row_rel_err(logits.cpu().numpy(), ref) <= LOGIT_TOL
        # the GPU's own selection is exactly the rule applied to the GPU's own logits ...
        assert np.array_equal(toks.cpu().numpy(), E.greedy_tokens(logits.cpu().numpy().astype(np.float64)))
        assert np.array_equal(toks.cpu().numpy(), toks2.cpu().numpy())
        # ... and agrees with the oracle wherever floating point leaves no doubt
        exact = check_tokens(toks.cpu().numpy(), ref)
        assert exact >= M // 2


def test_tokens_to_tokens_through_a_tiny_stage():
    """Embedding -> prefill of the 2-layer stage -> head on each prompt's last row -> one decode
    step fed by the selected tokens -> head: the chain a full pipeline runs, against the oracle."""
    sh = W.SHAPES["tiny"]
    vocab = 512
    lens = W.prefill_seq_lens("tiny", 4)
    pb = W.make_prefill_batch(lens + 1)
    cu = np.zeros(5, dtype=np.int32)
    cu[1:] = np.cumsum(lens)
    T = int(lens.sum())
    ids = W.token_ids(vocab, T, 3)
    with Ends(sh, vocab, max(T, 4)) as e, Stage(tdp, sh, pb.num_pages, 4, T, 4, pb.tables.shape[1]) as st:
        st.poison()
        x = torch.empty((T, sh.d_model), dtype=torch.bfloat16, device="cuda")
        tdp.tdp_embed_tokens(e.h, i32(ids), T, x)
        hid = torch.empty_like(x)
        tab = i32(pb.tables)
        tdp.tdp_stage_prefill(st.h, x, i32(cu), tab, 4, T, hid)
        last = (cu[1:] - 1).astype(np.int32)
        tok1 = torch.empty(4, dtype=torch.int32, device="cuda")
        lg1 = torch.empty((4, vocab), dtype=torch.float32, device="cuda")
        tdp.tdp_lm_head(e.h, hid, T, i32(last), 4, lg1, tok1)
        xd = torch.empty((4, sh.d_model), dtype=torch.bfloat16, device="cuda")
        tdp.tdp_embed_tokens(e.h, tok1, 4, xd)                 # token ids stay on the device
        hd = torch.empty_like(xd)
        tdp.tdp_stage_decode(st.h, xd, i32(lens), tab, 4, hd)
        tok2 = torch.empty(4, dtype=torch.int32, device="cuda")
        lg2 = torch.empty((4, vocab), dtype=torch.float32, device="cuda")
        tdp.tdp_lm_head(e.h, hd, 4, None, 4, lg2, tok2)
        torch.cuda.synchronize()
        # oracle chain; the decode step is fed the GPU's first tokens so that a near-tie in step 1
        # cannot masquerade as an error in step 2
        layers = list(oracle_layers(sh))
        osh = oracle_shape(sh)
        table, head, gain = f64(e.table), f64(e.head), f64(e.gain)
        xs = E.embed(ids, table)
        ref_h, caches = O.stage_prefill([xs[cu[s]:cu[s + 1]] for s in range(4)], layers, osh)
        ref_last = np.stack([r[-1] for r in ref_h])
        ref_lg1 = E.final_logits(ref_last, gain, head, sh.rms_eps)
        assert row_rel_err(lg1.cpu().numpy(), ref_lg1) <= 2e-2
        check_tokens(tok1.cpu().numpy(), ref_lg1)
        xd_ref = E.embed(tok1.cpu().numpy(), table)
        assert np.array_equal(f64(xd), xd_ref)
        ref_hd, _ = O.stage_decode(list(xd_ref), caches, layers, osh)
        ref_lg2 = E.final_logits(np.stack(ref_hd), gain, head, sh.rms_eps)
        assert row_rel_err(lg2.cpu().numpy(), ref_lg2) <= 2e-2
        check_tokens(tok2.cpu().numpy(), ref_lg2)


def test_lm_head_at_llama_size_sampled():
    """70B-shaped ends at decode batch 512: vocabulary 32000, d_model 8192.  The oracle computes
    48 sampled rows in full (every logit of those rows)."""
    sh = W.SHAPES["70b_quarter"]
    vocab, M = 32000, 512
    with Ends(sh, vocab, M) as e:
        x = W.hidden_states(sh, M, 9, device="cuda")
        toks = torch.empty(M, dtype=torch.int32, device="cuda")
        logits = torch.empty((M, vocab), dtype=torch.float32, device="cuda")
        tdp.tdp_lm_head(e.h, x, M, None, M, logits, toks)
        torch.cuda.synchronize()
        rows = np.unique(np.concatenate([[0, 1, M - 2, M - 1], W.token_ids(M, 44, 2)]))
        head = f64(e.head)
        ref = E.final_logits(f64(x)[rows], f64(e.gain), head, sh.rms_eps)
        assert row_rel_err(logits[torch.from_numpy(rows).cuda().long()].cpu().numpy(), ref) <= LOGIT_TOL
        check_tokens(toks.cpu().numpy()[rows], ref)
        assert np.array_equal(toks.cpu().numpy()[:64], E.greedy_tokens(logits[:64].cpu().numpy().astype(np.float64)))


@pytest.mark.parametrize("vocab", [3996, 4000, 19996, 20000, 32000])  # rows below and from 4000 columns on, a whole number of tiles and not
@pytest.mark.parametrize("M", [1, 33, 200, 512])             # tiles of 32 to 256 rows, the last one partly filled
def test_greedy_tokens_of_the_head_are_those_of_its_logits(M, vocab):
    """Few distinct columns in random places: every row's largest logit lies in many pieces of the row at once.  Rows that hold a
    NaN give only NaN, rows of zeros only ties."""
    d = 64
    g = torch.Generator(device="cuda").manual_seed(M + vocab)
    which = torch.randint(0, 40, (vocab,), generator=g, device="cuda")
    head = torch.randn(d, 40, generator=g, device="cuda").to(torch.bfloat16)[:, which].contiguous()
    x = torch.randn(M, d, generator=g, device="cuda").to(torch.bfloat16)
    x[M // 2, 5] = float("nan")
    x[M // 3] = 0
    h = tdp.tdp_ends_create(tdp.EndsConfig(vocab, d, 1e-5, M))
    tdp.tdp_ends_set_weight(h, tdp.E_LM_HEAD, head, tdp.BF16, tdp.DEVICE, d, vocab)
    tdp.tdp_ends_set_weight(h, tdp.E_FINAL_NORM, torch.ones(d, device="cuda"), tdp.F32, tdp.DEVICE, d, 1)
    logits = torch.empty((M, vocab), dtype=torch.float32, device="cuda")
    toks = torch.full((M,), -1, dtype=torch.int32, device="cuda")
    tdp.tdp_lm_head(h, x, M, None, M, logits, toks)
    torch.cuda.synchronize()
    tdp.tdp_ends_destroy(h)
    lg = logits.cpu().numpy().astype(np.float64)
    assert np.array_equal(toks.cpu().numpy(), E.greedy_tokens(np.where(np.isnan(lg), -np.inf, lg)))


@pytest.mark.parametrize("M", [3, 200])
def test_infinite_logits(M):
    """The first weight of chosen columns is minus infinity: their logits are minus infinity, infinity or (a zero in the hidden state)
    NaN by the sign of a row's first element.  All columns of the first half, every third one behind it; in the second vocabulary all."""
    d, vocab = 64, 4100
    g = torch.Generator(device="cuda").manual_seed(M)
    x = torch.randn(M, d, generator=g, device="cuda").to(torch.bfloat16)
    x[0, 0], x[1, 0], x[2, 0] = 1.0, -1.0, 0.0
    for columns in (torch.cat([torch.arange(vocab // 2), torch.arange(vocab // 2, vocab, 3)]), torch.arange(vocab)):
        head = torch.randn(d, vocab, generator=g, device="cuda").to(torch.bfloat16)
        head[0, columns.cuda()] = -float("inf")
        h = tdp.tdp_ends_create(tdp.EndsConfig(vocab, d, 1e-5, M))
        tdp.tdp_ends_set_weight(h, tdp.E_LM_HEAD, head, tdp.BF16, tdp.DEVICE, d, vocab)
        tdp.tdp_ends_set_weight(h, tdp.E_FINAL_NORM, torch.ones(d, device="cuda"), tdp.F32, tdp.DEVICE, d, 1)
        logits = torch.empty((M, vocab), dtype=torch.float32, device="cuda")
        toks = torch.full((M,), -1, dtype=torch.int32, device="cuda")
        tdp.tdp_lm_head(h, x, M, None, M, logits, toks)
        torch.cuda.synchronize()
        tdp.tdp_ends_destroy(h)
        lg = logits.cpu().numpy().astype(np.float64)
        up = x[:, 0].float().cpu().numpy() > 0
        assert np.isneginf(lg[up][:, columns]).all() and np.isnan(lg[2, columns]).all()
        assert np.array_equal(toks.cpu().numpy(), E.greedy_tokens(np.where(np.isnan(lg), -np.inf, lg)))
