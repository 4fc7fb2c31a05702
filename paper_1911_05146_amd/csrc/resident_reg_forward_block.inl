// Block bi of k_reg_forward (kernels_resident_reg.hip), included there in the loop over identity blocks and, with LD set, for the block that leads the
// run in, whose conv1 is behind it (acc0).  As a lambda for both the training kernel of the identity runs measured 0.6 % slower (other registers).
const bool more = bi + 1 < a.nblk;
const ResBlock B = a.blocks[bi];
const ResBlock Bn = a.blocks[more ? bi + 1 : bi];
const int ahead = INFER ? block_ahead(LD, bi, 2, a.nblk) : 0;
if constexpr (INFER) { if (!LD || ahead >= 0) next_offsets(ahead, bi + 1); }
// ---- conv1 (1x1, C -> MID) on relu(bn1(x))
floatx4 acc[RG_PTW][NM];
if constexpr (!INFER) w3.issue(a.packed + B.wf_off[2], wave, fr, fq);
if constexpr (LD) {
#pragma unroll
  for (int j = 0; j < RG_PTW; ++j)
#pragma unroll
    for (int nt = 0; nt < NM; ++nt) acc[j][nt] = acc0[j][nt];
} else {
#pragma unroll
  for (int j = 0; j < RG_PTW; ++j)
#pragma unroll
    for (int nt = 0; nt < NM; ++nt) acc[j][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < C / 32; ++ks) {
    bf16x8 bf[RG_PTW];
#pragma unroll
    for (int j = 0; j < RG_PTW; ++j)
      bf[j] = frag_of(bn_relu_pack(X[j][2 * ks], coefC + 2 * ks * 16 + fq * 4), bn_relu_pack(X[j][2 * ks + 1], coefC + (2 * ks + 1) * 16 + fq * 4));
#pragma unroll
    for (int nt = 0; nt < NM; ++nt) {
      const bf16x8 wf = W1::get(w1r, ks, nt);
#pragma unroll
      for (int j = 0; j < RG_PTW; ++j) acc[j][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, bf[j], acc[j][nt], 0, 0, 0);
    }
  }
}
uint2 cp[RG_PTW][NM];
#pragma unroll
for (int j = 0; j < RG_PTW; ++j)
#pragma unroll
  for (int nt = 0; nt < NM; ++nt) { cp[j][nt] = pack4(acc[j][nt]); acc[j][nt] = unpack4(cp[j][nt]); }
if constexpr (!INFER) {
  if (!exchange(IM{}, acc, B, 1, coefM, [&] {
        w3.commit(sW3, wave, lane);
        if constexpr (!WHOLE) { if (bi > 0) w2.template commit<2>(sW2, wave, lane); }
        px_store<MID != 32>(image(B.c1_off, MID), offM, cp);
      }))
    return;
}
#pragma unroll
for (int j = 0; j < RG_PTW; ++j)
#pragma unroll
  for (int nt = 0; nt < NM; ++nt)
    *reinterpret_cast<uint2*>(cv_w + j * RG_CW * MS + nt * 16) = bn_relu_pack(acc[j][nt], coefM + nt * 16 + fq * 4);
__syncthreads();
if constexpr (INFER) {   // every wave is past conv1 and its tables, and past conv3 of the block before
  w3.commit(sW3, wave, lane);
  if (!LD || ahead >= 0) {
    w1.commit(sW1, wave, lane);
    store_coef();
    load_coef();
    w1.issue(a.packed + nx.w1, wave, fr, fq);   // a whole block ahead of their use
    w3.issue(a.packed + nx.w3, wave, fr, fq);
  }
}
// ---- conv2 (3x3, MID -> MID)
#pragma unroll
for (int j = 0; j < RG_PTW; ++j)
#pragma unroll
  for (int nt = 0; nt < NM; ++nt) acc[j][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
conv3x3_rows<MID, false, W2>(cv_r, w2r, acc);
#pragma unroll
for (int j = 0; j < RG_PTW; ++j)
#pragma unroll
  for (int nt = 0; nt < NM; ++nt) { cp[j][nt] = pack4(acc[j][nt]); acc[j][nt] = unpack4(cp[j][nt]); }
if constexpr (INFER) {
  __syncthreads();
  if (!LD || ahead >= 0) {
    w2.commit(sW2, wave, lane);
    w2.issue(a.packed + nx.w2, wave, fr, fq);
  }
} else {
  auto next_w12 = [&] { w2.template issue<0>(a.packed + Bn.wf_off[1], wave, fr, fq); w1.issue(a.packed + Bn.wf_off[0], wave, fr, fq); };
  if constexpr (!WHOLE) { if (more) next_w12(); }   // the exchange hides it
  if (!exchange(IM{}, acc, B, 2, coefM3, [&] {
        if constexpr (WHOLE) { if (more) next_w12(); }
        else if (more) { w2.template commit<0>(sW2, wave, lane); w2.template issue<1>(a.packed + Bn.wf_off[1], wave, fr, fq); }
        px_store<MID != 32>(image(B.c2_off, MID), offM, cp);
      }))
    return;
}
// ---- conv3 (1x1, MID -> C) on relu(bn3(c2)), accumulated onto x
{
  bf16x8 bf[RG_PTW][MID / 32];
#pragma unroll
  for (int ks = 0; ks < MID / 32; ++ks)
#pragma unroll
    for (int j = 0; j < RG_PTW; ++j)
      bf[j][ks] = frag_of(bn_relu_pack(acc[j][2 * ks], coefM3 + 2 * ks * 16 + fq * 4), bn_relu_pack(acc[j][2 * ks + 1], coefM3 + (2 * ks + 1) * 16 + fq * 4));
#pragma unroll
  for (int nt = 0; nt < NC; ++nt)
#pragma unroll
    for (int ks = 0; ks < MID / 32; ++ks) {
      const bf16x8 wf = W3::get(w3r, ks, nt);
#pragma unroll
      for (int j = 0; j < RG_PTW; ++j) X[j][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, bf[j][ks], X[j][nt], 0, 0, 0);
    }
}
uint2 yp[RG_PTW][NC];
#pragma unroll
for (int j = 0; j < RG_PTW; ++j)
#pragma unroll
  for (int nt = 0; nt < NC; ++nt) { yp[j][nt] = pack4(X[j][nt]); X[j][nt] = unpack4(yp[j][nt]); }
auto store_y = [&] { px_store<MID != 32>(image(B.y_off, C), offC, yp); };
if constexpr (INFER) {
  if (!more) store_y();
} else if (more) {
  if (!exchange(IC{}, X, Bn, 0, coefC, [&] {
        w1.commit(sW1, wave, lane);
        if constexpr (WHOLE) w2.template commit<0>(sW2, wave, lane);
        else { w2.template commit<1>(sW2, wave, lane); w2.template issue<2>(a.packed + Bn.wf_off[1], wave, fr, fq); }
        store_y();
      }))
    return;
} else {
  store_y();
}
