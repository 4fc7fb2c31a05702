// Block bi of k_reg_backward (kernels_resident_reg.hip), included there in the loop over identity blocks and, with LD set, for the block that leads the
// run in (resident_reg_forward_block.inl).
using LP = LeadPx<C>;
constexpr int CI = LP::CI, NI = LP::NI;
using WL1 = WStage<CI, MID>;   // conv1 data gradient [CI][MID]
using WLP = WStage<CI, C>;     // projection data gradient [CI][C], staged where the canvas was
static_assert(WLP::BYTES <= RG_CW * RG_CW * MS * 2 && WL1::BYTES <= W1::BYTES, "the lead's matrices lie where the canvas and conv1's were");
const LP lp(row0, fr, fq);
WL1 l1;
WLP lw;
uint2 dcp[RG_PTW][NM], xe[RG_PTW][NI], xo[3 * RG_PTW][NI];   // xo: the pixels that only BatchNorm 1 reads
const ResBlock B = a.blocks[bi];
const bool more = !LD && bi > 0;
const ResBlock Bn = a.blocks[more ? bi - 1 : 0];
// ---- conv3 data gradient, BN3 + ReLU backward -> dc2
floatx4 acc[RG_PTW][NM];
#pragma unroll
for (int j = 0; j < RG_PTW; ++j)
#pragma unroll
  for (int nt = 0; nt < NM; ++nt) acc[j][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
if constexpr (LD) { l1.issue(a.packed + B.wd_off[0], wave, fr, fq); lw.issue(a.packed + B.pd_off, wave, fr, fq); }
else w1.issue(a.packed + B.wd_off[0], wave, fr, fq);
#pragma unroll
for (int ks = 0; ks < C / 32; ++ks)
#pragma unroll
  for (int nt = 0; nt < NM; ++nt) {
    const bf16x8 wf = W3::get(w3r, ks, nt);
#pragma unroll
    for (int j = 0; j < RG_PTW; ++j)
      acc[j][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, frag_of(DY[j][2 * ks], DY[j][2 * ks + 1]), acc[j][nt], 0, 0, 0);
  }
px_arrange(xc2);
if (!exchange(IM{}, std::bool_constant<LD>{}, acc, xc2, cf3, B, 2, [&] {
      if constexpr (LD) l1.commit(sW13, wave, lane);
      else w1.commit(sW13, wave, lane);   // every wave is past conv3's data gradient
      if (bi + 1 < a.nblk) w2.template commit<2>(sW2, wave, lane);
      if (bi + 1 < a.nblk) px_store<MID == 32>(image(a.blocks[bi + 1].gx_off, C), offC, DY);   // the gradient of the input of the block above
      px_load(xc1, image(B.c1_off, MID), offM);
      if constexpr (!LD) px_load(xx, image(B.x_off, C), offC);
    }))
  return;
#pragma unroll
for (int nt = 0; nt < NM; ++nt)
#pragma unroll
  for (int j = 0; j < RG_PTW; ++j) {
    dcp[j][nt] = pack4(bwd_apply<MID>(acc[j][nt], xc2[j][nt], tab + nt * 16 + fq * 4));
    *reinterpret_cast<uint2*>(cv_w + j * RG_CW * MS + nt * 16) = dcp[j][nt];
  }
__syncthreads();
// ---- conv2 data gradient, BN2 + ReLU backward -> dc1
#pragma unroll
for (int j = 0; j < RG_PTW; ++j)
#pragma unroll
  for (int nt = 0; nt < NM; ++nt) acc[j][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
conv3x3_rows<MID, true, W2>(cv_r, w2r, acc);
if (more) w2.template issue<0>(a.packed + Bn.wd_off[1], wave, fr, fq);   // every piece has an exchange to arrive
px_arrange(xc1);
if (!exchange(IM{}, std::bool_constant<LD>{}, acc, xc1, cf2, B, 1, [&] {
      if (more) { w2.template commit<0>(sW2, wave, lane); w2.template issue<1>(a.packed + Bn.wd_off[1], wave, fr, fq); }   // every wave is past conv2's data gradient
      px_store<MID == 32>(image(B.dc2_off, MID), offM, dcp);
      if (more) { load_tables(bi - 1); w3.issue(a.packed + Bn.wd_off[2], wave, fr, fq); }
      if constexpr (LD) {
        lw.commit(canvas, wave, lane);   // every wave is past conv2's data gradient
        const bf16_t* const x = cx.tensor(B.x_off) + (size_t)me * (4 * RG_P * CI);
#pragma unroll
        for (int t = 0; t < RG_LT; ++t) lp.load(t & 3 ? xo[t - 1 - (t >> 2)] : xe[t >> 2], x, t);
      }
    }))
  return;
#pragma unroll
for (int nt = 0; nt < NM; ++nt)
#pragma unroll
  for (int j = 0; j < RG_PTW; ++j) dcp[j][nt] = pack4(bwd_apply<MID>(acc[j][nt], xc1[j][nt], tab + nt * 16 + fq * 4));
if constexpr (LD) {
  // ---- conv1's and the projection's data gradients, BN1 + ReLU backward
  floatx4 da[RG_PTW][NI];
#pragma unroll
  for (int nt = 0; nt < NI; ++nt) {
#pragma unroll
    for (int j = 0; j < RG_PTW; ++j) da[j][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < MID / 32; ++ks) {
      const bf16x8 wf = WL1::get(w1r, ks, nt);
#pragma unroll
      for (int j = 0; j < RG_PTW; ++j)
        da[j][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, frag_of(dcp[j][2 * ks], dcp[j][2 * ks + 1]), da[j][nt], 0, 0, 0);
    }
#pragma unroll
    for (int ks = 0; ks < C / 32; ++ks) {
      const bf16x8 wf = WLP::get(canvas + lane * 8, ks, nt);
#pragma unroll
      for (int j = 0; j < RG_PTW; ++j)
        da[j][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, frag_of(DY[j][2 * ks], DY[j][2 * ks + 1]), da[j][nt], 0, 0, 0);
    }
  }
#pragma unroll
  for (int j = 0; j < RG_PTW; ++j) LP::arrange(xe[j]);
  if (!exchange(std::integral_constant<int, CI>{}, std::bool_constant<LD>{}, da, xe, cf1, B, 0, [&] {
        px_store<MID == 32>(image(B.dc1_off, MID), offM, dcp);
#pragma unroll
        for (int t = 0; t < 3 * RG_PTW; ++t) LP::arrange(xo[t]);
      }))
    return;
  bf16_t* const gx = cx.tensor(B.gx_off) + (size_t)me * (4 * RG_P * CI);
#pragma unroll
  for (int t = 0; t < RG_LT; ++t) {
    uint2 o[NI];
#pragma unroll
    for (int nt = 0; nt < NI; ++nt)
      o[nt] = pack4(bwd_apply<CI>(t & 3 ? floatx4{0.f, 0.f, 0.f, 0.f} : da[t >> 2][nt], t & 3 ? xo[t - 1 - (t >> 2)][nt] : xe[t >> 2][nt], tab + nt * 16 + fq * 4));
    lp.store(gx, t, o);
  }
} else {
  if constexpr (MID >= 64) px_store<MID == 32>(image(B.dc1_off, MID), offM, dcp);   // 16 registers that the exchange below cannot spare
  // ---- conv1 data gradient, BN1 + ReLU backward, plus the shortcut
  floatx4 da[RG_PTW][NC];
#pragma unroll
  for (int nt = 0; nt < NC; ++nt) {
#pragma unroll
    for (int j = 0; j < RG_PTW; ++j) da[j][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < MID / 32; ++ks) {
      const bf16x8 wf = W1::get(w1r, ks, nt);
#pragma unroll
      for (int j = 0; j < RG_PTW; ++j)
        da[j][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, frag_of(dcp[j][2 * ks], dcp[j][2 * ks + 1]), da[j][nt], 0, 0, 0);
    }
    if (nt % 4 == 3) keep_order();
  }
  px_arrange(xx);
  if (!exchange(IC{}, std::bool_constant<LD>{}, da, xx, cf1, B, 0, [&] {
        if (more) { w3.commit(sW13, wave, lane); w2.template commit<1>(sW2, wave, lane); w2.template issue<2>(a.packed + Bn.wd_off[1], wave, fr, fq); store_tables(); px_load(xc2, image(Bn.c2_off, MID), offM); }   // conv1's data gradient and the tables of this block are behind the barrier
        if constexpr (MID < 64) px_store<MID == 32>(image(B.dc1_off, MID), offM, dcp);
      }))
    return;
#pragma unroll
  for (int nt = 0; nt < NC; ++nt) {
    if (nt % 2 == 0) keep_order();
#pragma unroll
    for (int j = 0; j < RG_PTW; ++j)
      DY[j][nt] = pack4(bwd_apply<C>(da[j][nt], xx[j][nt], tab + nt * 16 + fq * 4) + unpack4(DY[j][nt]));
  }
}
