"""Child process of tests/test_gpu_ffn_schedule.py: micro-batches on streams
that may use only a few compute units, against the oracle and bit for bit
against the null stream.  The masked streams are created first (each takes a
hardware queue) and torch creates no stream here."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))


def main():
    import numpy as np
    import torch

    import oracle
    from paper_2606_22541_amd import inputs
    from paper_2606_22541_amd import moe_stage as C
    from paper_2606_22541_amd.stage import ExpertStage, bf16_bits, quantize_fp8, to_device_routing
    from gpu_common import BF16_TOL, FP8_TOL, check_outputs

    torch.cuda.set_device(0)
    C.load_library()
    streams = {n: C.moe_stream_create_cu_masked(0, n) for n in (16, 32)}
    for dtype in ("bf16", "fp8"):
        cfg = inputs.MoEConfig("few", d=512, f=256, E=16, e0=0, E_loc=5, k=4, lengths=(1300,), dtype=dtype,
                               has_shared=True, seed=91)
        wts = inputs.make_weights(cfg, "cuda")
        mb = inputs.make_microbatches(cfg, "cuda")[0]
        ids, w = to_device_routing(mb.ids, mb.w)
        x, xs = quantize_fp8(mb.x) if dtype == "fp8" else (mb.x, None)
        ref = oracle.run_stage(cfg, oracle.OracleWeights(wts, dtype), bf16_bits(mb.x), mb.ids, mb.w)
        with ExpertStage(cfg, wts) as st:
            outs = []
            for s in (0, streams[16], streams[32]):
                out = torch.full((1300, cfg.d), float("nan"), dtype=torch.bfloat16, device="cuda")
                m = st.microbatch(x, ids, w, out, xs)
                torch.cuda.synchronize()
                st.submit(m, s)
                st.sync()
                torch.cuda.synchronize()
                outs.append(bf16_bits(out))
                check_outputs(outs[-1], ref, FP8_TOL if dtype == "fp8" else BF16_TOL, "%s %s" % (dtype, s))
                print("%s on %s CUs ok" % (dtype, {0: "all"}.get(s, "a few")), flush=True)
            assert all(np.array_equal(outs[0], o) for o in outs[1:])
    for s in streams.values():
        C.moe_stream_destroy(s)
    print("FEW CUS OK", flush=True)


if __name__ == "__main__":
    main()
