import math
def growth(q,eta,m=4*math.pi):
    s=math.sinh
    b=[m*x for x in q]
    return b[0]*s(eta)+b[1]/2*s(2*eta)+b[2]/4*(s(3*eta)+3*s(eta))+b[3]/8*(s(4*eta)+4*s(2*eta))
for K in (8,12,16):
  for extra in (0,2):
    for eta in (2.2,2.5,2.7,3,3.5,4,5):
        B=(K-extra)*eta-math.log(4/(1e-15*(math.exp(eta)-1)))
        if B>0: print(K,extra,eta,'budget',round(B,2),'q1 max turns',round(B/(4*math.pi*math.sinh(eta)),5),'q2',round(B/(2*math.pi*math.sinh(2*eta)),6))
